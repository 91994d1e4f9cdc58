// The frame of a lane whose working set fits in LDS ("light" frames: at the usual operating
// points nearly all of them).
//
// What a frame computes is the paper's Section 3 / Fig. 1 sequence (emitting expansion with one
// thread per arc, adaptive beam, non-emitting iterations to convergence, contraction, lattice
// preprocessing of Section 3.4) - the same as the general frame.  How it is laid out differs,
// because at a few hundred tokens per lane a frame is not limited by bandwidth but by its
// chain of dependent steps, and this form is built to shorten that chain:
//   * the kept tokens of a frame stay in LDS (state handle, cost, position of their first
//     emitting arc) and are the next frame's queue, so a frame starts without any global read;
//     which token an arc belongs to is one LDS read: a bit marks every token's first arc, and
//     the token's number is the count of such bits up to the arc;
//   * every arc record carries the out-degrees of its destination, so a token is expanded
//     without fetching its state's header;
//   * all emitting arcs are expanded in one round, so the cutoff is final before the first
//     insertion: every state that enters the table is a kept token (unless max-active binds),
//     numbers itself when it is claimed, and no contraction step is needed; the candidates
//     stay in registers for the lattice stage;
//   * the closure works with one thread per epsilon arc: a claimed (or improved) state lists
//     its epsilon arcs in LDS, the next round fetches and relaxes the listed arcs side by side.
//     (Fetching them in the claiming thread, a state's arcs one after the other, made the
//     insertion and every round as long as the largest out-degree of a wave.);
//   * whatever is allotted (token numbers, arc positions, epsilon entries; lattice records) is
//     allotted once per wave: a DPP scan and one LDS atomic, not one per candidate;
//   * the per-frame counters come in two sets used alternately and the clearing of the state
//     table is deferred into the next frame's first stage, so a frame has three workgroup
//     barriers plus one per closure round, all of them LDS-only (global stores keep
//     travelling across them);
//   * a kept token is written to the channel's history exactly once, by the thread that holds
//     the candidate equal to the table's minimum (its best incoming arc), with the
//     back-pointer already in it.
// What bounds it: the chain of dependent steps (barriers, LDS and L2 round trips) and, with two
// lanes on a unit, the issue of its instructions.  Measured per frame, whole calls: 1 stream on the
// 8M-state graph at beam 13 (690 arcs a frame) 7.3 us, 300 frames on the 1000-state graph (2 270 arcs)
// 10.4 us, 500 streams 13.2 us.  With one thread per state in the closure, a contraction step and
// one allotment per candidate these took 12.5, 16.4 and 17.0 us.  In a build with timers (9.0 us for
// the first): start 1.1, expansion 1.6, insertion 1.4, closure 3.0 (2.3 rounds), history and lattice 1.6.
// Part of the issue is moves: a kernel that holds the three forms of a frame has more uniform values
// than scalar registers, and the compiler keeps 221 to 243 of them in lanes of vector registers (338
// with teams); v_readlane and v_writelane are 12 to 14 % of its vector instructions (16 % with teams).
// A frame that outgrows the LDS structures, or meets a state whose out-degrees do not fit the
// degree info, is redone in the heavy form or, where that one does not fit either, in the general
// one; nothing has been committed at that point.
#pragma once
#include <type_traits>
#include "wfst_lane.h"

namespace wfst {

// Prefix counts of the first-arc marks (see LaneShared::mark), by one whole wave.
template <int WORDS>
__device__ __forceinline__ void count_marks(uint2 *mark, uint32_t n_arcs) {
  constexpr int PER = WORDS / 64;
  const int lane = threadIdx.x & 63;
  if (n_arcs <= 64u * 32u) {                   // one word per lane
    const int inc = wave_incl_scan(__popc(mark[lane].x));
    mark[lane].y = (uint32_t)(inc - __popc(mark[lane].x));
    return;
  }
  int sum = 0, c[PER];
#pragma unroll
  for (int q = 0; q < PER; ++q) { c[q] = __popc(mark[lane * PER + q].x); sum += c[q]; }
  int run = wave_incl_scan(sum) - sum;
#pragma unroll
  for (int q = 0; q < PER; ++q) { mark[lane * PER + q].y = (uint32_t)run; run += c[q]; }
}

// Returns false if the frame must be redone in another form.
template <int NT>
__device__ __forceinline__ bool light_frame(const DecDev &D, LaneShared<NT> &S, LaneCtx &ctx, const float *ll, const float *ll_next,
                            bool is_init, int chan) {
  using L = LightCfg<NT>;
  constexpr int U = L::TILE / NT;
  constexpr uint32_t mask = L::SLOTS - 1;
  constexpr int hbits = L::HBITS;
  constexpr uint32_t NOSLOT = 0xFFFFu;
  int tid = threadIdx.x;
  // (hidden from the compiler, which would otherwise compute every tid-dependent index and
  // address once, before the loop over the frames, and keep them all in scratch memory)
  asm volatile("" : "+v"(tid));
  const int lane = tid & 63, wid = uni(tid >> 6);
  const unsigned long long below = (1ull << lane) - 1ull;
  const uint32_t *rec = D.g.rec;
  Slot *slots = S.table;
  const Slot fresh{~0ull, EMPTY, 0xFFFFFFFFu};
  FrameCtr &C = S.fc[ctx.par];
  uint2 *const mark_in = S.mark[ctx.par ^ 1], *const mark_out = S.mark[ctx.par];
  const int nf = ctx.nf;                       // index of the frame being written
  const long long out_base = ctx.hist_used;
  const int n_in = is_init ? 0 : ctx.n_in;
  const uint32_t sink = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) float *)S.sink;
  // (the lane's buffers are addressed from the decoder's arrays where they are used: eight
  // pointers less to keep in registers across the whole kernel)
  HTok *const hist = D.hist + (size_t)chan * (size_t)D.hist_cap;
  LatInt *const lat = D.lat + (size_t)chan * (size_t)D.lat_cap;
  const uint32_t claim_limit = min((uint32_t)L::CLAIM_LIMIT, (uint32_t)D.tokcap);

  // ---- 0. what the previous light frame left: its table entries are cleared here, while this frame's
  //         first memory round trip is under way (cleared before it: a dictation's 360 frames and
  //         12 partial results take 3.98 instead of 3.94 ms) --------------------------------------
  uint32_t to_clear = ctx.pending_clear;
  ctx.pending_clear = 0;
  auto clear_table = [&]() {
#pragma unroll 1
    for (uint32_t i = tid; i < to_clear; i += NT) slots[S.lq[i]] = fresh;
    to_clear = 0;
  };
  if (nf > D.max_frames) { ctx.status = E_HISTORY_OVERFLOW; return true; }
  if (!is_init && !ctx.tok_valid) {            // the token list is not in LDS (first frame of a call, or after a general frame)
    clear_table();
#pragma unroll 1
    for (int w = tid; w < L::MARK_WORDS; w += NT) { mark_in[w] = make_uint2(0, 0); mark_out[w] = make_uint2(0, 0); }
    if (tid == 0) S.list_dead = 0;
    if (ctx.lds_foreign) {
#pragma unroll 1
      for (int i = tid; i < L::SLOTS; i += NT) slots[i] = fresh;
      ctx.lds_foreign = false;
    }
    lds_barrier();
    uint32_t base = 0;
#pragma unroll 1
    for (int tb = 0; tb < n_in; tb += NT) {
      const int i = tb + tid;
      int a = 0;                               // arc positions the token takes (one if it has no emitting arc)
      if (i < n_in) {
        const HTok t = hist[ctx.hist_used - n_in + i];
        const uint32_t h = t.handle & HMASK, ne = rec[3 * (size_t)h];
        S.tok[i] = make_uint2(h | (ne ? 0u : TOK_DEAD), __float_as_uint(t.cost));
        if (!ne) atomicAdd(&S.list_dead, 1u);
        a = (int)min(max(ne, 1u), (uint32_t)L::ARCS + 1u);
      }
      const int inc = wave_incl_scan(a);
      if (lane == 63) S.wtot[wid] = inc;
      lds_barrier();
      uint32_t pos = base + (uint32_t)(inc - a);
#pragma unroll
      for (int w = 0; w < NT / 64; ++w) { const int t = uni(S.wtot[w]); pos += w < wid ? t : 0; base += (uint32_t)t; }
      if (i < n_in) {
        S.tok_a[i] = (uint16_t)pos;
        if (pos < (uint32_t)L::ARCS) atomicOr(&mark_in[pos >> 5].x, 1u << (pos & 31));
      }
      lds_barrier();
    }
    if (base > (uint32_t)L::ARCS) return false;
    if (wid == 0) count_marks<L::MARK_WORDS>(mark_in, base);
    ctx.n_arcs = base; ctx.n_dead = uni(S.list_dead);
    ctx.tok_valid = true;
    lds_barrier();
  }
  const int total = is_init ? 0 : (int)ctx.n_arcs;
  if (total > L::ARCS || (total > L::TILE && L::TILE * 5 / 4 > D.auxcap)) { clear_table(); ctx.tok_valid = false; __syncthreads(); return false; }   // (the barrier: the table is clear before the next light frame)

  PHASE_MARK(0);
  // A claimed state takes the frame's next token number, that many arc positions for the next
  // frame and lists its epsilon arcs.  False if one of the structures is full.
  auto put = [&](uint32_t sl, uint32_t dw, uint32_t info, uint32_t ci, uint32_t apos, uint32_t e0) -> bool {
    const uint32_t ne = info & INFO_NE, np = info >> INFO_NP_SHIFT, h = dw & HMASK;
    // (out-degrees too large for the info: the general frame reads the header)
    if (ci >= claim_limit || e0 + np > (uint32_t)L::ECAP || ne == INFO_NE || np == INFO_NP) return false;
    S.lq[ci] = (uint16_t)sl;
    S.tok[ci].x = h | (ne ? 0u : TOK_DEAD);
    S.tok_a[ci] = (uint16_t)apos;
    slots[sl].aux = (info << 16) | ci;
    if (apos < (uint32_t)L::ARCS) atomicOr(&mark_out[apos >> 5].x, 1u << (apos & 31));
    if (!ne) atomicAdd(&C.dead, 1u);
#pragma unroll 1
    for (uint32_t k = 0; k < np; ++k) { S.ea_r[e0 + k] = h + 1 + ne + k; S.ea_s[e0 + k] = (uint16_t)sl; }
    return true;
  };

  // ---- 1. emitting expansion ------------------------------------------------------------------
  // Arc u * NT + tid of a tile is this thread's u-th.  A frame of one tile (nearly all are) takes 1,
  // 2 or 4 slots per thread, whatever is enough, in straight-line code: the look-ups of all slots
  // side by side, then all record loads, then all score loads; its candidates stay in registers.
  // Of a frame of two tiles the second is expanded first and its candidates wait in global memory,
  // each thread its own, until the cutoff is known (the insertion overwrites the token list).
  float x[U]; uint32_t r[U], nsk[U];           // cost, arc, slot of the destination | source token << 16
  uint32_t dw[U], kx[U], w2[U];
  Aux *const notes = D.aux + (size_t)blockIdx.x * (size_t)D.auxcap;
  auto expand = [&](auto slots_per_thread, int tile) {
    constexpr int UA = decltype(slots_per_thread)::value;
    float wt[UA], ct[UA], sc[UA];
    int j[UA], have[UA];
    uint2 m[UA], t[UA];
    uint32_t k[UA], a0[UA];
    // (a lane past the end re-reads the last arc, so that no load is conditional)
#pragma unroll
    for (int u = 0; u < UA; ++u) { j[u] = min(tile * L::TILE + u * NT + tid, total - 1); m[u] = mark_in[j[u] >> 5]; }
#pragma unroll
    for (int u = 0; u < UA; ++u) k[u] = m[u].y + (uint32_t)__popc(m[u].x & ((2u << (j[u] & 31)) - 1u)) - 1u;
#pragma unroll
    for (int u = 0; u < UA; ++u) { t[u] = S.tok[k[u]]; a0[u] = S.tok_a[k[u]]; }
#pragma unroll
    for (int u = 0; u < UA; ++u) {
      // (a token without an emitting arc: its state's header is read and nothing done with it)
      const uint32_t dead = t[u].x >> 31;
      r[u] = (t[u].x & HMASK) + 1u + (uint32_t)j[u] - a0[u] - dead;
      ct[u] = __uint_as_float(t[u].y);
      have[u] = (int)(tile * L::TILE + u * NT + tid < total) & (int)(dead ^ 1u);
      nsk[u] = NOSLOT | (k[u] << 16);
      const uint32_t *a = rec + 3 * (size_t)r[u];
      dw[u] = a[0]; wt[u] = __uint_as_float(a[1]); w2[u] = a[2];
    }
    __builtin_amdgcn_sched_barrier(0);         // (keeps the loads above together and their uses below them)
    clear_table();
#pragma unroll
    for (int u = 0; u < UA; ++u) sc[u] = ll[have[u] ? w2[u] & D.g.pdf_mask : 0u];
    __builtin_amdgcn_sched_barrier(0);
    int bad = 0;
#pragma unroll
    for (int u = 0; u < UA; ++u) {
      x[u] = (ct[u] + wt[u]) - sc[u];
      const int fine = (int)(x[u] > -INFINITY);                  // (neither NaN nor -inf)
      bad |= have[u] & (fine ^ 1);
      kx[u] = (have[u] & fine) ? okey(x[u]) : KEY_NONE;
    }
    if (bad) C.flags = F_NAN;                  // (the only flag that this stage sets)
  };
  auto best_of = [&](auto slots_per_thread) {
    constexpr int UA = decltype(slots_per_thread)::value;
    uint32_t best = KEY_NONE;
#pragma unroll
    for (int u = 0; u < UA; ++u) best = min(best, kx[u]);
    best = wave_min_u32(best);
    if (lane == 0 && best != KEY_NONE) atomicMin(&C.best, best);
  };
  // ---- 2. insertion of the candidates within the cutoff ------------------------------------------
  auto insert = [&](auto slots_per_thread, float cut) {
    constexpr int UA = decltype(slots_per_thread)::value;
    uint32_t hs[UA], got[UA];                  // slot looked at, and what it held
    uint32_t wanted = 0, open = 0;             // slots u with a candidate; ... whose place in the table is not found yet
#pragma unroll
    for (int u = 0; u < UA; ++u) {
      hs[u] = slot_hash(dw[u] & HMASK, hbits);
      got[u] = EMPTY;
      if (kx[u] != KEY_NONE && x[u] <= cut) {
        wanted |= 1u << u;
        got[u] = atomicCAS(&slots[hs[u]].handle, EMPTY, dw[u] & HMASK);
      }
    }
#pragma unroll
    for (int u = 0; u < UA; ++u) open |= (got[u] != EMPTY && got[u] != (dw[u] & HMASK)) ? 1u << u : 0u;
#pragma unroll 1
    for (uint32_t tries = 1; open && tries < L::MAX_PROBES; ++tries) {
#pragma unroll
      for (int u = 0; u < UA; ++u) {
        if (open & (1u << u)) {
          hs[u] = (hs[u] + slot_step(dw[u] & HMASK)) & mask;
          got[u] = atomicCAS(&slots[hs[u]].handle, EMPTY, dw[u] & HMASK);
        }
      }
#pragma unroll
      for (int u = 0; u < UA; ++u) if (got[u] == EMPTY || got[u] == (dw[u] & HMASK)) open &= ~(1u << u);
    }
    bool full = open != 0;
    wanted &= ~open;
    uint32_t n_new = 0, n_eps = 0, n_arc = 0;
#pragma unroll
    for (int u = 0; u < UA; ++u) {
      if (wanted & (1u << u)) {
        atomicMin(&slots[hs[u]].val, pack(kx[u], r[u]));
        nsk[u] = (nsk[u] & 0xFFFF0000u) | hs[u];
      }
      const bool is_new = (wanted & (1u << u)) && got[u] == EMPTY;
      n_new += is_new ? 1u : 0u;
      n_eps += is_new ? w2[u] >> (16 + INFO_NP_SHIFT) : 0u;
      n_arc += is_new ? max((w2[u] >> 16) & INFO_NE, 1u) : 0u;
    }
    if (__ballot(n_new != 0)) {
      const uint32_t inc = (uint32_t)wave_incl_scan((int)(n_new | (n_eps << 16))), inca = (uint32_t)wave_incl_scan((int)n_arc);
      unsigned long long base = 0;
      if (lane == 63) base = atomicAdd(&C.cnt[0], ((unsigned long long)inca << CNT_ARC_SHIFT) | inc);
      const uint32_t b0 = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)base, 63);
      uint32_t apos = ((uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(base >> CNT_ARC_SHIFT), 63) & CNT_ARCS) + inca - n_arc;
      uint32_t ci = (b0 & 0xFFFFu) + (inc & 0xFFFFu) - n_new, e0 = (b0 >> 16) + (inc >> 16) - n_eps;
#pragma unroll
      for (int u = 0; u < UA; ++u) {
        if ((wanted & (1u << u)) && got[u] == EMPTY) {
          if (!put(hs[u], dw[u], w2[u] >> 16, ci, apos, e0)) full = true;
          ++ci; apos += max((w2[u] >> 16) & INFO_NE, 1u); e0 += w2[u] >> (16 + INFO_NP_SHIFT);
        }
      }
    }
    if (full) atomicOr(&C.cnt[0], CNT_RESTART);
  };
  auto first_tile = [&](auto slots_per_thread) {
    expand(slots_per_thread, 0);
    best_of(slots_per_thread);
    lds_barrier();
    PHASE_MARK(2);
    const uint32_t bk = C.best, fl = C.flags;
    if (!(uni(fl) & F_NAN)) insert(slots_per_thread, key2f(uni(bk)) + D.beam);   // (the cutoff is final here)
  };
  constexpr std::integral_constant<int, U> whole{};
  const bool two_tiles = total > L::TILE;
  const int ua = (total + NT - 1) / NT;        // slots that are enough
  const bool has_arcs = total > wid * 64;      // a wave without arcs skips all this
  uint32_t *const note_src = reinterpret_cast<uint32_t *>(notes + L::TILE);
  if (two_tiles) {
    expand(whole, 1);
    best_of(whole);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      notes[u * NT + tid] = Aux{dw[u], kx[u] == KEY_NONE ? __builtin_nanf("") : x[u], r[u], w2[u]};
      note_src[u * NT + tid] = nsk[u];
    }
  }
  if (is_init) {
    if (tid == 0) {
      C.best = okey(0.0f);
      const uint32_t h = D.g.start_handle;
      const uint32_t sl = slot_hash(h, hbits);               // (the table is empty)
      slots[sl].handle = h; slots[sl].val = pack(okey(0.0f), NO_ARC);
      const uint32_t ne = D.g.start_info & INFO_NE, np = (D.g.start_info >> INFO_NP_SHIFT) & INFO_NP;
      C.cnt[0] = ((unsigned long long)max(ne, 1u) << CNT_ARC_SHIFT) | ((unsigned long long)np << CNT_EPS_SHIFT) | 1ull;
      if (!put(sl, h, D.g.start_info, 0u, 0u, 0u)) C.cnt[0] |= CNT_RESTART;
    }
  } else if (!has_arcs) {
    clear_table();
    lds_barrier();
  } else if (ua == 1) {
    first_tile(std::integral_constant<int, 1>{});
  } else if (ua == 2) {
    first_tile(std::integral_constant<int, 2>{});
  } else {
    first_tile(whole);
  }
  if (two_tiles) {
    float x0[U]; uint32_t r0[U], nsk0[U];      // (the first tile's candidates)
#pragma unroll
    for (int u = 0; u < U; ++u) { x0[u] = x[u]; r0[u] = r[u]; nsk0[u] = nsk[u]; }
    const uint32_t bk = C.best, fl = C.flags;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const Aux a = notes[u * NT + tid];
      dw[u] = a.slot; x[u] = a.x; r[u] = a.arc; w2[u] = a.src; kx[u] = okey(a.x); nsk[u] = note_src[u * NT + tid];
    }
    if (!(uni(fl) & F_NAN)) insert(whole, key2f(uni(bk)) + D.beam);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      notes[u * NT + tid] = Aux{nsk[u], x[u], r[u], 0u};
      x[u] = x0[u]; r[u] = r0[u]; nsk[u] = nsk0[u];
    }
  }
  lds_barrier();
  PHASE_MARK(3);
  if (tid == 0) reset_ctr(S.fc[ctx.par ^ 1]);  // the previous frame's counters: nobody reads them any more
#pragma unroll 1
  for (int w = tid; w < L::MARK_WORDS; w += NT) mark_in[w] = make_uint2(0, 0);      // (read in stage 1 only)

  const uint32_t bestk = uni(C.best);
  const unsigned long long c0 = uni(C.cnt[0]);
  int abort_code = 0;                          // 1: give the frame to the general form
  {
    const uint32_t fl = uni(C.flags);
    if (c0 & CNT_RESTART) abort_code = 1;
    else if (fl & F_NAN) abort_code = E_NAN_INPUT;
    else if (bestk == KEY_NONE || bestk == KEY_PINF) abort_code = E_DEAD_CHANNEL;
  }
  const float cutoff = key2f(bestk) + D.beam;
  // fetch ahead the next frame's row of scores (one 64-byte line per load): by the next
  // expansion its gathers by pdf id hit L2
  if (ll_next) {
#pragma unroll 1
    for (int p = tid * 16; p < D.g.num_pdfs; p += NT * 16) fetch_ahead(ll_next + p, sink);
  }

  // ---- 3. non-emitting closure ----------------------------------------------------------------
  // Round k relaxes the epsilon arcs listed in the round before, each from its source's current
  // cost.  What round k lists is counted by counter (k + 1) % 3, which nobody touches in round
  // k + 1, so one barrier per round is enough.
  uint32_t e_lo = 0, e_hi = (uint32_t)(c0 >> CNT_EPS_SHIFT) & 0xFFFFu;
  uint32_t nclaim = (uint32_t)c0 & 0xFFFFu, narcs = (uint32_t)(c0 >> CNT_ARC_SHIFT) & CNT_ARCS;
  int iters = 0;
  while (abort_code == 0 && e_lo < e_hi) {
    unsigned long long *ctr = &C.cnt[(iters + 1) % 3];
    if (tid == 0) C.cnt[(iters + 2) % 3] = 0;
#pragma unroll 1
    for (uint32_t i0 = e_lo + wid * 64; i0 < e_hi; i0 += NT) {
      const uint32_t i = min(i0 + lane, e_hi - 1);
      const uint32_t re = S.ea_r[i], src = S.ea_s[i] & EA_SLOT;
      const uint32_t *a = rec + 3 * (size_t)re;
      const uint32_t dw = a[0]; const float w = __uint_as_float(a[1]); const uint32_t w2 = a[2];
      const float xe = key2f(reinterpret_cast<const uint32_t *>(&slots[src].val)[1]) + w;
      const uint32_t h = dw & HMASK, info = w2 >> 16;
      uint32_t sl = slot_hash(h, hbits);
      bool is_new = false, again = false, full = false;
      const bool mine = i0 + lane < e_hi;
      if (mine && xe <= cutoff) {
        uint32_t got, tries = 0;
#pragma unroll 1
        for (;;) {
          got = atomicCAS(&slots[sl].handle, EMPTY, h);
          if (got == EMPTY || got == h || ++tries >= L::MAX_PROBES) break;
          sl = (sl + slot_step(h)) & mask;
        }
        if (got == EMPTY || got == h) {
          const unsigned long long old = atomicMin(&slots[sl].val, pack(okey(xe), re));
          is_new = got == EMPTY;
          again = !is_new && (dw & HAS_EPS) && okey(xe) < (uint32_t)(old >> 32);     // its epsilon arcs must be relaxed once more
        } else {
          full = true;
        }
      } else {
        sl = NOSLOT;
      }
      if (mine) { S.ea_w[i] = w; S.ea_d[i] = (uint16_t)sl; }
      const unsigned long long m_new = __ballot(is_new);
      if (m_new | __ballot(again)) {
        const uint32_t np = info >> INFO_NP_SHIFT;
        const uint32_t v = (is_new ? max(info & INFO_NE, 1u) : 0u) | ((is_new || again) ? np << 20 : 0u);
        const uint32_t inc = (uint32_t)wave_incl_scan((int)v);
        unsigned long long base = 0;
        if (lane == 63)
          base = atomicAdd(ctr, ((unsigned long long)(inc & 0xFFFFFu) << CNT_ARC_SHIFT) | ((unsigned long long)(inc >> 20) << CNT_EPS_SHIFT) |
                                    (unsigned long long)__popcll(m_new));
        const uint32_t b0 = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)base, 63);
        const uint32_t ba = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(base >> CNT_ARC_SHIFT), 63) & CNT_ARCS;
        const uint32_t ex = inc - v;
        const uint32_t e0 = e_hi + (b0 >> 16) + (ex >> 20);
        if (is_new) {
          if (!put(sl, dw, info, nclaim + (b0 & 0xFFFFu) + (uint32_t)__popcll(m_new & below), narcs + ba + (ex & 0xFFFFFu), e0)) full = true;
        } else if (again) {
          const uint32_t ne = info & INFO_NE;
          if (ne == INFO_NE || np == INFO_NP || e0 + np > (uint32_t)L::ECAP) full = true;
          else {
            atomicAdd(&C.again, np);
#pragma unroll 1
            for (uint32_t k = 0; k < np; ++k) { S.ea_r[e0 + k] = h + 1 + ne + k; S.ea_s[e0 + k] = (uint16_t)(sl | EA_AGAIN); }
          }
        }
      }
      if (full) atomicOr(ctr, CNT_RESTART);
    }
    lds_barrier();
    const unsigned long long cv = uni(*ctr);   // stable: the next round lists through another counter
    e_lo = e_hi; e_hi += (uint32_t)(cv >> CNT_EPS_SHIFT) & 0xFFFFu;
    nclaim += (uint32_t)cv & 0xFFFFu; narcs += (uint32_t)(cv >> CNT_ARC_SHIFT) & CNT_ARCS;
    ++iters;
    if (cv & CNT_RESTART) abort_code = 1;
  }
  if (abort_code == 1) {                       // outgrew the LDS structures: wipe the table, the heavy or the general frame redoes it
    // (Every wave has read the counters by now, not only the first one, which resets them: a wave that
    // came late would find no request to give up, take the frame for done and be a barrier off from then on.)
    lds_barrier();
#pragma unroll 1
    for (int i = tid; i < L::SLOTS; i += NT) slots[i] = fresh;
    if (tid == 0) reset_ctr(C);
    ctx.tok_valid = false;
    __syncthreads();
#ifdef WFST_PHASE_TIMING
    if (tid == 0) S.ph[13] += 1;
#endif
    PHASE_MARK(14);
    return false;
  }
  PHASE_MARK(4);

  // ---- 4. max-active selection ------------------------------------------------------------------
  // Only if more states than max_active were reached: the kept ones are numbered anew.
  float cutoff_eff = cutoff;
  uint32_t n_out = abort_code == 0 ? nclaim : 0u;
  uint32_t n_valid = n_out;                    // tokens within the beam
  if (abort_code == 0) {
    const uint32_t room = (uint32_t)min((long long)0x7FFFFFFF, D.hist_cap - out_base);
    if ((D.approximate ? nclaim : min(nclaim, (uint32_t)D.max_active)) > room) { abort_code = E_HISTORY_OVERFLOW; n_out = 0; n_valid = 0; }
    else if (nclaim > (uint32_t)D.max_active) {
      auto key_of = [&](int i) { return reinterpret_cast<const uint32_t *>(&slots[S.lq[i]].val)[1]; };
      uint32_t kmin = 0xFFFFFFFFu, kmax = 0;
#pragma unroll 1
      for (int i = tid; i < (int)nclaim; i += NT) { const uint32_t k = key_of(i); kmin = min(kmin, k); kmax = max(kmax, k); }
      kmin = wave_min_u32(kmin); kmax = ~wave_min_u32(~kmax);
      if (lane == 0) { atomicMin(&C.kmin, kmin); atomicMax(&C.kmax, kmax); }
#pragma unroll 1
      for (int w = tid; w < L::MARK_WORDS; w += NT) mark_out[w] = make_uint2(0, 0);
      __syncthreads();
      const int n = (int)nclaim;
      uint32_t theta, h_theta = 0xFFFFFFFFu;                  // keep key < theta, or == theta with handle <= h_theta
      auto by_key = [&](int i, uint32_t &v) { v = key_of(i); return true; };
      if (D.approximate) {
        theta = block_histogram_cut<NT>(S, n, (uint32_t)D.max_active, uni(C.kmin), uni(C.kmax), by_key);   // (every key <= theta is kept)
      } else {
        uint32_t n_less, n_eq;
        block_select<NT>(S, n, (uint32_t)D.max_active, uni(C.kmin), uni(C.kmax), by_key, theta, n_less, n_eq);
        const uint32_t need_eq = (uint32_t)D.max_active - n_less;
        if (need_eq < n_eq) {
          uint32_t hl, he;
          block_select<NT>(S, n, need_eq, 0u, HMASK,
                           [&](int i, uint32_t &v) {
                             if (key_of(i) != theta) return false;
                             v = slots[S.lq[i]].handle;
                             return true;
                           }, h_theta, hl, he);
        }
      }
      cutoff_eff = key2f(theta);
      if (tid == 0) { C.dead = 0; C.sel = 0; }
      __syncthreads();
#pragma unroll 1
      for (int i0 = wid * 64; i0 < n; i0 += NT) {
        const int i = min(i0 + lane, n - 1);
        const uint32_t sl = S.lq[i];
        const Slot sv = ld_slot<true>(slots + sl);
        const uint32_t key = (uint32_t)(sv.val >> 32), info = sv.aux >> 16, ne = info & INFO_NE;
        const bool keep = i0 + lane < n && (key < theta || (key == theta && sv.handle <= h_theta));
        const unsigned long long m = __ballot(keep);
        const uint32_t na = keep ? max(ne, 1u) : 0u, inc = (uint32_t)wave_incl_scan((int)na);
        unsigned long long base = 0;
        if (lane == 63 && m) base = atomicAdd(&C.sel, ((unsigned long long)inc << 32) | (unsigned long long)__popcll(m));
        const uint32_t pos = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)base, 63) + (uint32_t)__popcll(m & below);
        const uint32_t apos = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(base >> 32), 63) + inc - na;
        if (keep) {
          S.tok[pos].x = sv.handle | (ne ? 0u : TOK_DEAD); S.tok_a[pos] = (uint16_t)apos;
          if (apos < (uint32_t)L::ARCS) atomicOr(&mark_out[apos >> 5].x, 1u << (apos & 31));
          if (!ne) atomicAdd(&C.dead, 1u);
        }
        if (i0 + lane < n) slots[sl].aux = (info << 16) | (keep ? pos : POS_NONE);
      }
      lds_barrier();
      const unsigned long long sel = uni(C.sel);
      n_out = (uint32_t)sel; narcs = (uint32_t)(sel >> 32);
    }
  }
  PHASE_MARK(8);

  // ---- 5. history records, back-pointers and lattice records ---------------------------------
  // Every candidate arc is looked at once more, with final costs.  The one equal to the table's
  // minimum is the token's best incoming arc: its thread writes the token's history record.
  // Every arc into a kept token within the effective cutoff and the lattice beam is recorded
  // with its extra cost (Section 3.4).
  if (abort_code == 0) {
    const long long lat_base = ctx.lat_pos, lat_room = D.lat_cap - ctx.lat_pend;
    auto emit_lat = [&](uint32_t p, uint32_t arc, float extra, uint32_t dst, uint32_t src) {
      if ((long long)p >= lat_room) atomicOr(&C.flags, F_LATOVF);
      else {
        long long at = lat_base + (long long)p;
        if (at >= D.lat_cap) at -= D.lat_cap;
        lat[at] = LatInt{nf, arc, extra, dst, src};
      }
    };
    // the token `pos` gets its history record and its cost in the LDS list
    auto finish = [&](uint32_t pos, const Slot &sv, float cost, uint32_t arc, uint32_t prev) {
      hist[out_base + pos] = HTok{sv.handle | ((sv.aux >> (16 + INFO_NP_SHIFT)) ? HAS_EPS : 0u), cost, arc, prev};
      S.tok[pos].y = __float_as_uint(cost);
    };
    auto finish_emitting = [&](auto slots_per_thread) {
      constexpr int UA = decltype(slots_per_thread)::value;
      Slot sv[UA];
#pragma unroll
      for (int u = 0; u < UA; ++u) sv[u] = ld_slot<true>(slots + min(nsk[u] & 0xFFFFu, mask));
      uint32_t rec_mask = 0, n_rec = 0;
#pragma unroll
      for (int u = 0; u < UA; ++u) {
        const uint32_t pos = sv[u].aux & POS_NONE;
        const bool kept = (nsk[u] & 0xFFFFu) != NOSLOT && pos != POS_NONE;
        if (kept && pack(okey(x[u]), r[u]) == sv[u].val) finish(pos, sv[u], x[u], r[u], nsk[u] >> 16);
        const float extra = x[u] - key2f((uint32_t)(sv[u].val >> 32));
        const bool wanted = kept && D.lattice_on && x[u] <= cutoff_eff && extra <= D.lattice_beam;
        x[u] = extra;
        nsk[u] = (nsk[u] & 0xFFFF0000u) | pos;
        rec_mask |= wanted ? 1u << u : 0u;
        n_rec += (uint32_t)__popcll(__ballot(wanted));
      }
      if (n_rec) {
        uint32_t p = 0;
        if (lane == 0) p = atomicAdd(&C.latn, n_rec);
        p = uni(p);
#pragma unroll
        for (int u = 0; u < UA; ++u) {
          const bool wanted = rec_mask & (1u << u);
          const unsigned long long m = __ballot(wanted);
          if (wanted) emit_lat(p + (uint32_t)__popcll(m & below), r[u], x[u], nsk[u] & 0xFFFFu, nsk[u] >> 16);
          p += (uint32_t)__popcll(m);
        }
      }
    };
    if (!has_arcs) { }
    else if (ua == 1) finish_emitting(std::integral_constant<int, 1>{});
    else if (ua == 2) finish_emitting(std::integral_constant<int, 2>{});
    else {
#pragma unroll 1
      for (int tile = 0;; ++tile) {
        finish_emitting(whole);
        if (tile > 0 || !two_tiles) break;
#pragma unroll
        for (int u = 0; u < U; ++u) { const Aux a = notes[u * NT + tid]; nsk[u] = a.slot; x[u] = a.x; r[u] = a.arc; }
      }
    }
#pragma unroll 1
    for (uint32_t i0 = wid * 64; i0 < e_hi; i0 += NT) {
      const uint32_t i = min(i0 + lane, e_hi - 1);
      const uint32_t es = S.ea_s[i], re = S.ea_r[i];
      uint32_t dsl = S.ea_d[i];
      const Slot ssv = ld_slot<true>(slots + (es & EA_SLOT));
      const uint32_t spos = ssv.aux & POS_NONE;
      const float xe = key2f((uint32_t)(ssv.val >> 32)) + S.ea_w[i];
      float extra = 0.f;
      uint32_t pos = POS_NONE;
      bool wanted = false;
      if (i0 + lane < e_hi && !(es & EA_AGAIN) && xe <= cutoff_eff) {
        if (dsl == NOSLOT) {                     // beyond the cutoff when first relaxed, within it after its source improved
          const int f = ht_find<true>(slots, mask, hbits, rec[3 * (size_t)re] & HMASK);
          dsl = f < 0 ? NOSLOT : (uint32_t)f;
        }
        if (dsl != NOSLOT) {
          const Slot sv = ld_slot<true>(slots + dsl);
          pos = sv.aux & POS_NONE;
          if (pos != POS_NONE) {
            // a best incoming arc whose source was cut by max-active leaves the token without a
            // back-pointer (a best path through it reports a broken trace)
            if (pack(okey(xe), re) == sv.val) finish(pos, sv, xe, re, spos == POS_NONE ? NO_ARC : (spos | PREV_SAME));
            extra = xe - key2f((uint32_t)(sv.val >> 32));
            wanted = D.lattice_on && spos != POS_NONE && extra <= D.lattice_beam;
          }
        }
      }
      const unsigned long long m = __ballot(wanted);
      if (m) {
        uint32_t p = 0;
        if (lane == 0) p = atomicAdd(&C.latn, (uint32_t)__popcll(m));
        p = uni(p);
        if (wanted) emit_lat(p + (uint32_t)__popcll(m & below), re, extra, pos, spos | PREV_SAME);
      }
    }
    if (is_init && tid == 0) {                 // the start token has no incoming arc
      const int sl = ht_find<true>(slots, mask, hbits, D.g.start_handle);
      const uint32_t pos = sl >= 0 ? (slots[sl].aux & POS_NONE) : POS_NONE;
      if (pos != POS_NONE && (uint32_t)slots[sl].val == NO_ARC) finish(pos, slots[sl], 0.0f, NO_ARC, NO_ARC);
    }
    if (wid == NT / 64 - 1) count_marks<L::MARK_WORDS>(mark_out, narcs);     // for the next frame's expansion
  }
  lds_barrier();
  PHASE_MARK(9);

  // ---- 6. the lane's state after the frame (every thread computes the same values) -----------
  const uint4 ends = *reinterpret_cast<const uint4 *>(&C.flags);   // flags, latn, dead, again
  if (abort_code == 0 && (uni(ends.x) & F_LATOVF)) abort_code = E_LATTICE_OVERFLOW;
  const long long lat_new = min((long long)uni(ends.y), D.lat_cap - ctx.lat_pend);
  if (tid == NT - 1) {                         // (of the wave least likely to have had arcs)
    (D.frame_off + (size_t)chan * (size_t)(D.max_frames + 2))[nf + 1] = out_base + n_out;
    S.arcs_expanded += (long long)(total - (is_init ? 0 : (int)ctx.n_dead)) + (n_valid ? (long long)(e_hi - ends.w) : 0ll);
    S.max_pre = max(S.max_pre, (int)n_valid);
    S.max_post = max(S.max_post, (int)n_out);
    S.iters_max = max(S.iters_max, iters);
  }
  ctx.nf = nf + 1;
  ctx.n_in = (int)n_out;
  ctx.n_arcs = narcs; ctx.n_dead = uni(ends.z);
  ctx.hist_used = out_base + n_out;
  ctx.lat_total += lat_new; ctx.lat_pend += lat_new;
  ctx.lat_pos += lat_new;
  if (ctx.lat_pos >= D.lat_cap) ctx.lat_pos -= D.lat_cap;
#ifdef WFST_PHASE_TIMING
  if (tid == 0) { S.ph[7] += iters; S.dbg_tok += n_out; }
#endif
  if (abort_code != 0) ctx.status = abort_code;
  ctx.tok_valid = abort_code == 0;
  ctx.pending_clear = nclaim;
  ctx.par ^= 1;
  return true;
}

}  // namespace wfst
