// The general form of a lane's frame (any size, any graph).
#pragma once
#include "wfst_lane.h"

namespace wfst {

// One frame of one lane in its general form: state table, token queue and candidate notes in
// the lane's global scratch, tokens and state headers read from memory.  It handles frames of
// any size (up to the decoder's capacities) and every graph; what fits the LDS forms takes those
// (wfst_frame_light.h, wfst_frame_heavy.h).  Stages as listed at the top of wfst_kernels.h.
// (Inputs hidden from the compiler, as the heavy frame's.)
template <int NT, bool TEAM>
__device__ __forceinline__ void general_frame(ConstDev *Dp, int my_lane, int chan, const float *ll, int is_init) {
  asm volatile("" : "+s"(Dp), "+s"(my_lane), "+s"(chan));
  ConstDev &D = *(ConstDev *)uni((unsigned long long)Dp);
  LaneShared<NT> &S = lane_lds<NT, TEAM>();
  my_lane = uni(my_lane); chan = uni(chan); ll = uni(ll); is_init = uni(is_init);
  Slot *const gslots = D.slots + (size_t)my_lane * D.H;
  uint32_t *const queue = D.queue + (size_t)my_lane * (size_t)D.qcap;
  Aux *const aux = D.aux + (size_t)my_lane * (size_t)D.auxcap;
  uint32_t *const dkey = D.dkey + (size_t)my_lane * (size_t)D.tokcap, *const dslot = D.dslot + (size_t)my_lane * (size_t)D.tokcap;
  long long *const foff = D.frame_off + (size_t)chan * (size_t)(D.max_frames + 2);
  HTok *const hist = D.hist + (size_t)chan * (size_t)D.hist_cap;
  LatInt *const lat = D.lat + (size_t)chan * (size_t)D.lat_cap;
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  GenCtr &C = S.gen;
  const uint32_t *rec = D.g.rec;
  constexpr bool LDS = false;                // table words are read with coherent global loads
#ifdef WFST_PHASE_TIMING
  if (threadIdx.x == 0) S.gtlast = wall_clock64();
#endif
  Slot *slots = gslots;
  const uint32_t mask = D.H - 1;
  const int hbits = D.hbits;
  const Slot fresh{~0ull, EMPTY, A_FRESH};

  if (tid == 0) {
    C.claim_ctr = 0; C.auxn = 0; C.best = KEY_NONE; C.flags = 0; C.nvalid = 0; C.nout = 0; C.latn = 0;
    C.kmin = 0xFFFFFFFFu; C.kmax = 0; C.emit_arcs = 0; C.eps_arcs = 0;
  }
  __syncthreads();
  const int nf = S.nf;                       // index of the frame being written
  const long long out_base = S.hist_used;
  int abort_code = 0;
  if (nf > D.max_frames) abort_code = E_HISTORY_OVERFLOW;

  // the frame's token queue: claimed slots, plus re-expansion requests for improved ones
  const uint32_t qcap = (uint32_t)D.qcap;
  auto qget = [&](uint32_t i, uint32_t &sl, bool &eps, bool &dup) {
    const uint32_t e = queue[i]; sl = e & Q_SLOT; eps = e & Q_EPS; dup = e & Q_DUP;
  };
  auto on_claim = [&](int sl, uint32_t dw, bool dup) {
    // the lanes of the wave that call this together get consecutive queue entries and, those
    // that claimed a new state, consecutive claim numbers, from a single 64-bit atomic add
    const unsigned long long m_all = __ballot(1), m_new = __ballot(!dup);
    const int wl = threadIdx.x & 63, leader = __ffsll((long long)m_all) - 1;
    unsigned long long base = 0;
    if (wl == leader) base = atomicAdd(&C.claim_ctr, ((unsigned long long)__popcll(m_new) << 32) | (unsigned long long)__popcll(m_all));
    base = __shfl(base, leader, 64);
    const unsigned long long below = (1ull << wl) - 1ull;
    if (!dup) {
      const uint32_t ci = (uint32_t)(base >> 32) + (uint32_t)__popcll(m_new & below);
      if (ci >= (uint32_t)D.tokcap) atomicOr(&C.flags, F_TOKOVF);
    }
    const uint32_t q = (uint32_t)base + (uint32_t)__popcll(m_all & below);
    if (q >= qcap) atomicOr(&C.flags, F_TOKOVF);
    else queue[q] = (uint32_t)sl | ((dw & HAS_EPS) ? Q_EPS : 0u) | (dup ? Q_DUP : 0u);
  };

  // ---- 1. emitting expansion ------------------------------------------------------------
  if (abort_code == 0) {
    if (is_init) {
      if (tid == 0) {
        const uint32_t h = D.g.start_handle;
        bool cl, im;
        const int sl = ht_insert<LDS>(slots, mask, hbits, h, pack(okey(0.0f), NO_ARC), cl, im);
        on_claim(sl, rec[3 * (size_t)h + 1] ? HAS_EPS : 0u, false);
        C.best = okey(0.0f);
      }
    } else {
      const long long in_off = S.in_off;
      const int n_in = S.n_in;
      // touch this frame's row of scores (one 64-byte line per thread) while the tokens'
      // graph records are being fetched, so that the gathers by pdf id below hit L2
      const float touch = tid * 16 < D.g.num_pdfs ? ll[tid * 16] : 0.f;
      float touch_more = 0.f;
      for (int p = (NT + tid) * 16; p < D.g.num_pdfs; p += NT * 16) touch_more += ll[p];
      // this thread's token of a tile: state handle, cost, emitting out-degree
      auto load_token = [&](int i, uint32_t &h, float &c, int &ne) {
        ne = 0; h = 0; c = 0.f;
        if (i < n_in) {
          const HTok t = hist[in_off + i];
          h = t.handle & HMASK; c = t.cost;
          ne = (int)rec[3 * (size_t)h];
        }
      };
      uint32_t h, hn = 0; float c, cn = 0.f; int ne, nen = 0;
      load_token(tid, h, c, ne);
      for (int tb = 0; tb < n_in; tb += NT) {
        int total;
        const int ex = block_excl_scan<NT, LDS>(ne, S.wave_tmp, total);
        S.scan[tid] = ex; S.cost[tid] = c; S.base[tid] = h + 1;
        wg_sync<LDS>();
        GEN_MARK(8);
        if (tid == 0) C.emit_arcs += (unsigned long long)total;
        if (tb + NT < n_in) load_token(tb + NT + tid, hn, cn, nen);   // next tile, in flight during this one's rounds
        // one thread per arc (Section 3.3), EXP_U arcs of the tile per thread and round so
        // that their loads are in flight together
        for (int j0 = 0; j0 < total; j0 += NT * EXP_U) {
          float x[EXP_U], ct[EXP_U], sll[EXP_U]; uint32_t r[EXP_U], dw[EXP_U], kx[EXP_U], wt[EXP_U], w2[EXP_U]; int kk[EXP_U];
          int lo[EXP_U], hi[EXP_U], jc[EXP_U];
          // (a lane past the end re-reads the tile's last arc, so that no load is conditional and all
          // record loads, then all score loads, of a round are in flight together)
#pragma unroll
          for (int u = 0; u < EXP_U; ++u) { jc[u] = min(j0 + u * NT + tid, total - 1); lo[u] = 0; hi[u] = NT - 1; }
          constexpr int STEPS = NT >= 1024 ? 10 : NT >= 512 ? 9 : 8;
#pragma unroll
          for (int it = 0; it < STEPS; ++it) {     // largest k with scan[k] <= j, the searches step by step side by side
            int v[EXP_U];
#pragma unroll
            for (int u = 0; u < EXP_U; ++u) v[u] = S.scan[(lo[u] + hi[u] + 1) >> 1];
#pragma unroll
            for (int u = 0; u < EXP_U; ++u) { const int mid = (lo[u] + hi[u] + 1) >> 1; if (v[u] <= jc[u]) lo[u] = mid; else hi[u] = mid - 1; }
          }
#pragma unroll
          for (int u = 0; u < EXP_U; ++u) {
            kk[u] = lo[u];
            r[u] = S.base[lo[u]] + (uint32_t)(jc[u] - S.scan[lo[u]]);
            ct[u] = S.cost[lo[u]];
          }
#pragma unroll
          for (int u = 0; u < EXP_U; ++u) {
            const uint32_t *a = rec + 3 * (size_t)r[u];
            dw[u] = a[0]; wt[u] = a[1]; w2[u] = a[2];
          }
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int u = 0; u < EXP_U; ++u) sll[u] = ll[w2[u] & D.g.pdf_mask];
          __builtin_amdgcn_sched_barrier(0);
          uint32_t m = KEY_NONE;
          bool bad = false;
#pragma unroll
          for (int u = 0; u < EXP_U; ++u) {
            x[u] = (ct[u] + __uint_as_float(wt[u])) - sll[u];
            const bool have = j0 + u * NT + tid < total;
            const bool nan = x[u] != x[u] || x[u] == -INFINITY;
            bad |= have && nan;
            kx[u] = (have && !nan) ? okey(x[u]) : KEY_NONE;
            m = min(m, kx[u]);
          }
          if (bad) atomicOr(&C.flags, F_NAN);
          m = wave_min_u32(m);
          if ((tid & 63) == 0 && m != KEY_NONE) atomicMin(&C.best, m);
          wg_sync<LDS>();
          GEN_MARK(9);
          const float cut = key2f(C.best) + D.beam;     // running bound, never below the final cutoff
#pragma unroll
          for (int u = 0; u < EXP_U; ++u) {
            if (kx[u] == KEY_NONE || !(x[u] <= cut)) continue;
            bool cl, im;
            const int sl = ht_insert<LDS>(slots, mask, hbits, dw[u] & HMASK, pack(kx[u], r[u]), cl, im);
            if (sl < 0) { atomicOr(&C.flags, F_TOKOVF); continue; }
            if (cl) on_claim(sl, dw[u], false);
            if (D.lattice_on || im) {
              const uint32_t ai = wave_alloc(&C.auxn);
              if (ai >= (uint32_t)D.auxcap) atomicOr(&C.flags, F_LATOVF);
              else aux[ai] = Aux{(uint32_t)sl, x[u], r[u], (uint32_t)(tb + kk[u])};
            }
          }
        }
        wg_sync<LDS>();
        GEN_MARK(10);
        h = hn; c = cn; ne = nen;
      }
      asm volatile("" ::"v"(touch), "v"(touch_more));
    }
  }
  __syncthreads();
  GEN_MARK(0);
  const uint32_t bestk = C.best;
  if (abort_code == 0) {
    const uint32_t fl = C.flags;
    if (fl & F_NAN) abort_code = E_NAN_INPUT;
    else if (fl & F_TOKOVF) abort_code = E_TOKEN_OVERFLOW;
    else if (fl & F_LATOVF) abort_code = E_LATTICE_OVERFLOW;
    else if (bestk == KEY_NONE || bestk == KEY_PINF) abort_code = E_DEAD_CHANNEL;
  }
  const float cutoff = key2f(bestk) + D.beam;

  // ---- 2. non-emitting closure ----------------------------------------------------------
  // One epsilon arc of an expanded token: note it for the lattice stage on the token's first
  // expansion (source slot, weight, arc, destination), then offer the candidate.
  auto relax_eps = [&](uint32_t src_slot, float c, uint32_t r, uint32_t dw, float w, uint32_t note_at) {
    if (note_at < (uint32_t)D.auxcap) aux[note_at] = Aux{src_slot | AUX_EPS, w, r, dw & HMASK};
    const float x = c + w;
    if (!(x <= cutoff)) return;
    bool cl, im;
    const int sl = ht_insert<LDS>(slots, mask, hbits, dw & HMASK, pack(okey(x), r), cl, im);
    if (sl < 0) { atomicOr(&C.flags, F_TOKOVF); return; }
    if (cl || im) on_claim(sl, dw, !cl);
  };
  int iters = 0;
  if (abort_code == 0) {
    uint32_t w0 = 0, w1 = min((uint32_t)C.claim_ctr, qcap);
    __syncthreads();
    while (w0 < w1) {
      // every thread takes CU queue entries of the window per pass, their loads side by side; the
      // pass is kept convergent (predicated, no early exit) so that the wave can allot note space
      // with one atomic
      constexpr int CU = 4;
      for (uint32_t i0 = w0; i0 < w1; i0 += NT * CU) {
        bool act[CU], first[CU]; uint32_t src[CU], h[CU], ne[CU], np[CU]; float c[CU]; Slot sv[CU];
#pragma unroll
        for (int u = 0; u < CU; ++u) {
          const uint32_t i = i0 + (uint32_t)u * NT + tid;
          act[u] = false; first[u] = false; src[u] = 0; h[u] = 0; ne[u] = 0; np[u] = 0; c[u] = 0.f;
          if (i < w1) {
            bool eps, dup;
            qget(i, src[u], eps, dup);
            act[u] = eps;
          }
        }
#pragma unroll
        for (int u = 0; u < CU; ++u) if (act[u]) sv[u] = ld_slot<LDS>(&slots[src[u]]);
#pragma unroll
        for (int u = 0; u < CU; ++u)
          if (act[u]) { c[u] = key2f((uint32_t)(sv[u].val >> 32)); act[u] = c[u] <= cutoff; h[u] = sv[u].handle; }
#pragma unroll
        for (int u = 0; u < CU; ++u) if (act[u]) { ne[u] = rec[3 * (size_t)h[u]]; np[u] = rec[3 * (size_t)h[u] + 1]; }
        uint32_t fr[CU];
#pragma unroll
        for (int u = 0; u < CU; ++u) fr[u] = act[u] ? atomicAnd(&slots[src[u]].aux, ~A_FRESH) : 0u;   // first expansion while within the cutoff
#pragma unroll
        for (int u = 0; u < CU; ++u) first[u] = (fr[u] & A_FRESH) != 0;
        uint32_t dwv[CU][EPS_U]; float wv[CU][EPS_U];                // the first arcs, loads in flight together
#pragma unroll
        for (int u = 0; u < CU; ++u)
#pragma unroll
          for (int k = 0; k < EPS_U; ++k) {
            dwv[u][k] = 0; wv[u][k] = 0.f;
            if (act[u] && (uint32_t)k < np[u]) {
              const uint32_t *a = rec + 3 * (size_t)(h[u] + 1 + ne[u] + k);
              dwv[u][k] = a[0]; wv[u][k] = __uint_as_float(a[1]);
            }
          }
        // note space and the arc count, one atomic per wave
        uint32_t nn = 0;
#pragma unroll
        for (int u = 0; u < CU; ++u) nn += first[u] ? np[u] : 0u;
        const uint32_t inc = (uint32_t)wave_incl_scan((int)nn);
        const uint32_t wave_total = (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
        uint32_t note = 0;
        if ((tid & 63) == 0 && wave_total) {
          note = atomicAdd(&C.auxn, wave_total);
          atomicAdd(&C.eps_arcs, (unsigned long long)wave_total);
          if (note + wave_total > (uint32_t)D.auxcap) atomicOr(&C.flags, F_LATOVF);
        }
        note = (uint32_t)__builtin_amdgcn_readlane((int)note, 0) + inc - nn;
#pragma unroll
        for (int u = 0; u < CU; ++u) {
#pragma unroll
          for (int k = 0; k < EPS_U; ++k)
            if (act[u] && (uint32_t)k < np[u]) relax_eps(src[u], c[u], h[u] + 1 + ne[u] + k, dwv[u][k], wv[u][k], first[u] ? note + k : 0xFFFFFFFFu);
          for (uint32_t k = EPS_U; act[u] && k < np[u]; ++k) {
            const uint32_t *a = rec + 3 * (size_t)(h[u] + 1 + ne[u] + k);
            relax_eps(src[u], c[u], h[u] + 1 + ne[u] + k, a[0], __uint_as_float(a[1]), first[u] ? note + k : 0xFFFFFFFFu);
          }
          if (first[u]) note += np[u];
        }
      }
      __syncthreads();
      GEN_MARK(11);
      w0 = w1; w1 = min((uint32_t)C.claim_ctr, qcap);
      ++iters;
      __syncthreads();
    }
    const uint32_t fl2 = C.flags;
    if (fl2 & F_TOKOVF) abort_code = E_TOKEN_OVERFLOW;
    else if (fl2 & F_LATOVF) abort_code = E_LATTICE_OVERFLOW;
  }
  GEN_MARK(1);
  const uint32_t n_q = min((uint32_t)C.claim_ctr, qcap);
  auto token_slot = [&](uint32_t i, uint32_t &sl, uint32_t &eps) -> bool {
    bool e, dup;
    qget(i, sl, e, dup);
    eps = e;
    return !dup;
  };

  // ---- 3 + 4. max-active selection and contraction into the token history ---------------
  float cutoff_eff = cutoff;
  if (abort_code == 0) {
    const uint32_t nclaim = (uint32_t)(C.claim_ctr >> 32);
    const uint32_t room = (uint32_t)min((long long)0x7FFFFFFF, D.hist_cap - out_base);
    if ((D.approximate ? nclaim : min(nclaim, (uint32_t)D.max_active)) > room) abort_code = E_HISTORY_OVERFLOW;
    else if (nclaim <= (uint32_t)D.max_active) {
      // nothing can be pruned: every token within the beam is kept
      for (uint32_t i = tid; i < n_q; i += NT) {
        uint32_t sl, eps;
        if (!token_slot(i, sl, eps)) continue;
        Slot *sp = slots + sl;
        const Slot sv = ld_slot<LDS>(sp);
        const unsigned long long v = sv.val;
        const float c = key2f((uint32_t)(v >> 32));
        if (!(c <= cutoff)) continue;
        const uint32_t pos = wave_alloc(&C.nout);
        if (pos >= room) continue;
        hist[out_base + pos] = HTok{sv.handle | (eps ? HAS_EPS : 0u), c, (uint32_t)v, NO_ARC};
        sp->aux = pos;
      }
      __syncthreads();
      if (tid == 0) C.nvalid = C.nout;
    } else {
      for (uint32_t i = tid; i < n_q; i += NT) {
        uint32_t sl, eps;
        if (!token_slot(i, sl, eps)) continue;
        const uint32_t key = (uint32_t)(tl64<LDS>(&slots[sl].val) >> 32);
        if (!(key2f(key) <= cutoff)) continue;
        const uint32_t p = wave_alloc(&C.nvalid);
        dkey[p] = key; dslot[p] = sl | (eps ? Q_EPS : 0u);
        atomicMin(&C.kmin, key); atomicMax(&C.kmax, key);
      }
      __syncthreads();
      const int n = (int)C.nvalid;
      const uint32_t kmin = C.kmin, kmax = C.kmax;
      uint32_t theta = KEY_NONE, h_theta = 0xFFFFFFFFu;       // keep key < theta, or == theta with handle <= h_theta
      auto by_key = [&](int i, uint32_t &v) { v = dkey[i]; return true; };
      auto by_handle_at_theta = [&](int i, uint32_t &v) {
        if (dkey[i] != theta) return false;
        v = tl32<LDS>(&slots[dslot[i] & Q_SLOT].handle);
        return true;
      };
      if (n > D.max_active && D.approximate) {
        theta = block_histogram_cut<NT>(S, n, (uint32_t)D.max_active, kmin, kmax, by_key);
        cutoff_eff = key2f(theta);                            // (every key <= theta is kept)
      } else if (n > D.max_active) {
        uint32_t n_less, n_eq;
        block_select<NT>(S, n, (uint32_t)D.max_active, kmin, kmax, by_key, theta, n_less, n_eq);
        const uint32_t need_eq = (uint32_t)D.max_active - n_less;
        if (need_eq < n_eq) {
          uint32_t hl, he;
          block_select<NT>(S, n, need_eq, 0u, HMASK, by_handle_at_theta, h_theta, hl, he);
        }
        cutoff_eff = key2f(theta);
      }
      for (uint32_t i = tid; i < (uint32_t)n; i += NT) {
        const uint32_t key = dkey[i], ds = dslot[i];
        Slot *sp = slots + (ds & Q_SLOT);
        const uint32_t h = tl32<LDS>(&sp->handle);
        const bool keep = key < theta || (key == theta && h <= h_theta);
        uint32_t pos = 0xFFFFFFFFu;
        if (keep) pos = wave_alloc(&C.nout);
        if (pos < room) {
          hist[out_base + pos] = HTok{h | ((ds & Q_EPS) ? HAS_EPS : 0u), key2f(key), (uint32_t)tl64<LDS>(&sp->val), NO_ARC};
          sp->aux = pos;
        } else {
          sp->aux = 0xFFFFFFFFu;
        }
      }
    }
  }
  __syncthreads();
  GEN_MARK(2);
  const uint32_t nout_all = C.nout;
  const uint32_t n_out = (abort_code == 0) ? (D.approximate ? nout_all : min(nout_all, (uint32_t)D.max_active)) : 0u;

  // ---- 5. lattice records and back-pointers ---------------------------------------------
  if (abort_code == 0) {
    const long long lat_base = S.lat_pos;
    const uint32_t n_aux = min(C.auxn, (uint32_t)D.auxcap);
    auto emit_lat = [&](uint32_t arc, float extra, uint32_t dst, uint32_t src) {
      const uint32_t p = wave_alloc(&C.latn);
      if ((long long)p >= S.lat_room) atomicOr(&C.flags, F_LATOVF);
      else {
        long long at = lat_base + (long long)p;
        if (at >= D.lat_cap) at -= D.lat_cap;
        lat[at] = LatInt{nf, arc, extra, dst, src};
      }
    };
    for (uint32_t i0 = 0; i0 < n_aux; i0 += NT * LAT_U) {
      Aux a[LAT_U];
#pragma unroll
      for (int u = 0; u < LAT_U; ++u) {
        const uint32_t i = i0 + (uint32_t)u * NT + tid;
        a[u] = i < n_aux ? aux[i] : Aux{0xFFFFFFFFu, 0.f, 0u, 0u};
      }
#pragma unroll
      for (int u = 0; u < LAT_U; ++u) {
        if (a[u].slot == 0xFFFFFFFFu) continue;
        if (!(a[u].slot & AUX_EPS)) {
          // emitting candidate {slot of the destination, x, arc, index of the source token}
          const Slot sv = ld_slot<LDS>(slots + a[u].slot);
          const uint32_t pos = sv.aux;
          if (pos >= A_KEPT_MAX) continue;
          const unsigned long long v = sv.val;
          if (pack(okey(a[u].x), a[u].arc) == v) hist[out_base + pos].prev = a[u].src;
          if (D.lattice_on && a[u].x <= cutoff_eff) {
            const float extra = a[u].x - key2f((uint32_t)(v >> 32));
            if (extra <= D.lattice_beam) emit_lat(a[u].arc, extra, pos, a[u].src);
          }
        } else {
          // epsilon arc {slot of the source | AUX_EPS, weight, arc, handle of the destination}
          const Slot ssv = ld_slot<LDS>(slots + (a[u].slot & ~AUX_EPS));
          const uint32_t spos = ssv.aux;
          if (spos >= A_KEPT_MAX) continue;                        // the source token was not kept
          const float x = key2f((uint32_t)(ssv.val >> 32)) + a[u].x;
          if (!(x <= cutoff_eff)) continue;
          const int sl = ht_find<LDS>(slots, mask, hbits, a[u].src);
          if (sl < 0) continue;
          const Slot sv = ld_slot<LDS>(slots + sl);
          const uint32_t pos = sv.aux;
          if (pos >= A_KEPT_MAX) continue;
          const unsigned long long v = sv.val;
          if (pack(okey(x), a[u].arc) == v) hist[out_base + pos].prev = spos | PREV_SAME;
          if (D.lattice_on) {
            const float extra = x - key2f((uint32_t)(v >> 32));
            if (extra <= D.lattice_beam) emit_lat(a[u].arc, extra, pos, spos | PREV_SAME);
          }
        }
      }
    }
  }
  __syncthreads();
  GEN_MARK(3);

  // ---- 6. clear the table ---------------------------------------------------------------
  const uint32_t fl3 = C.flags;
  if (fl3 & F_TOKOVF) {                                            // untracked claims: wipe everything
    const uint32_t n_all = D.H;
    for (uint32_t i = tid; i < n_all; i += NT) slots[i] = fresh;
  } else {
    for (uint32_t i = tid; i < n_q; i += NT) {
      uint32_t sl, eps;
      if (token_slot(i, sl, eps)) slots[sl] = fresh;
    }
  }
  if (tid == 0) {
    if (abort_code == 0 && (fl3 & F_LATOVF)) abort_code = E_LATTICE_OVERFLOW;
    const long long lat_new = min((long long)C.latn, S.lat_room);
    if (nf <= D.max_frames) {
      foff[nf + 1] = out_base + n_out;
      S.nf = nf + 1;
      S.in_off = out_base; S.n_in = (int)n_out;      // the frame just written is what the next one expands
    }
    S.hist_used = out_base + n_out;
    S.lat_total += lat_new; S.lat_room -= lat_new;
    S.lat_pos += lat_new;
    if (S.lat_pos >= D.lat_cap) S.lat_pos -= D.lat_cap;
    S.arcs_expanded += (long long)(C.emit_arcs + C.eps_arcs);
    S.max_pre = max(S.max_pre, (int)C.nvalid);
    S.max_post = max(S.max_post, (int)n_out);
    S.iters_max = max(S.iters_max, iters);
#ifdef WFST_PHASE_TIMING
    S.ph[7] += iters; S.dbg_tok += n_out; S.dbg_iters += iters; S.dbg_arcs += C.emit_arcs + C.eps_arcs;
#endif
    if (abort_code != 0) S.status = abort_code;
  }
  __syncthreads();
  GEN_MARK(4);
}

}  // namespace wfst
