// The frame of a lane that does not fit the light form: thousands of tokens, tens of thousands
// of arcs.  The state table is in LDS all the same - of one workgroup, or, when a call has so few
// lanes that the device would otherwise stand idle (Section 3.1: small batches are bound by
// latency), of up to sixteen workgroups that divide the states of a lane among them by hash: each
// owns its states' table entries, and candidates travel to their owner through buckets in global
// memory (every pair of workgroups has one of its own, so a bucket has one writer and one reader).
// What one workgroup would do between two of its barriers the team does between two team barriers:
//   1. expansion: every workgroup expands its share of the tokens; candidates within the best cost
//      it has seen + beam go to the owner's bucket;                                        barrier
//   2. insertion: the owner enters what is within the cutoff, now final, into its table; every
//      entered state is a token (unless max-active binds); states with epsilon arcs list them;
//   3. closure: a workgroup relaxes its listed epsilon arcs until it has none left, candidates for
//      other owners go to their buckets;                       barrier, and again until none was sent
//   4. max-active: histograms over (cost, state) pairs, added up in global memory;     barrier per pass
//      once few enough are left at the cut they are listed and ranked;                         barrier
//   5. every owner numbers its kept tokens, looks at its emitting candidates once more with final
//      costs (history records, lattice records), and sends its epsilon candidates;             barrier
//   6. the same for the epsilon candidates received;                                           barrier
// A frame that fills a table, a bucket or a list is given up, before anything is committed, and
// redone by the general frame.
//
// What bounds it: work inside a workgroup (LDS atomics and dependent loads per candidate) more than
// the team's barriers.  One stream of 42 000 arcs and up to 29 000 tokens per frame, team of eight,
// 73 us a frame: closure 29 (five to seven rounds), history and lattice 14, selection 9, arcs 7,
// insertion 5, tile lists and the barrier behind the expansion 3 each; about a dozen barriers of
// 1.1 - 1.5 us are a fifth of it.  (One workgroup: its table is too small for most of these frames,
// which become general: 487 us.  150 streams of 7 000 arcs a frame, the whole call divided by the 140
// frames of the longest (62 % of all frames are light): 102 us with one workgroup each, 65 with a second one
// for 104 of them, with the tables searched slot by slot; 62 now.)
// A team's workgroups are laid out on one XCD (the dispatcher deals workgroups to the eight XCDs in
// turn), whose L2 they share: a barrier then needs no write-back, only stores acknowledged by the
// L2, an arrival count and an invalidation of the vector cache.  Measured with 16 bytes stored per
// thread in front of each: 1.1 us for 8 workgroups, 1.7 us for 16; with device-scope release and
// acquire 2.0 and 3.1 us on one XCD, 1.4 and 1.6 us on several.  They check where they run; on
// several XCDs they use the latter.
#pragma once
#include "wfst_lane.h"

namespace wfst {

constexpr uint32_t TEAM_SPIN_LIMIT = 1u << 24;      // default number of polls before a barrier is given up (seconds)

// Returns false (to every thread of the workgroup) if a barrier of the team was given up: the
// workgroup must then stop working on the lane (what it would read may be incomplete).
template <int NT>
__device__ __forceinline__ bool team_sync(const TeamCtx &W, LaneShared<NT> &S) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wave's stores have been acknowledged
  __syncthreads();
  if (threadIdx.x == 0) {
    const uint32_t epoch = S.team.epoch + (uint32_t)W.G;
    S.team.epoch = epoch;
    bool ok = true;
    if (!W.same_xcd) __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    atomicAdd(&W.tl->arrived, 1u);
    uint32_t spins = 0;
    while ((int32_t)(ld32(&W.tl->arrived) - epoch) < 0) {
      if (++spins > W.spin_limit || ld32(&W.tl->broken)) { atomicExch(&W.tl->broken, 1u); ok = false; break; }
      __builtin_amdgcn_s_sleep(1);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    S.team_ok = ok ? 1u : 0u;
  }
  __syncthreads();
  return uni(S.team_ok) != 0;
}

template <int NT, bool TEAM>
__device__ __forceinline__ auto &heavy_counters(LaneShared<NT> &S, TeamCtx &W) {
  if constexpr (TEAM) return W.tl->ctr[W.seq & 1]; else return S.hc;
}
enum { HEAVY_DONE = 0, HEAVY_GIVEN_UP = 1, HEAVY_BROKEN = 2 };

// One frame; the lane's state is in S.hs (and, of the first workgroup, the rest of it in S).  The
// lane's scratch: aux / infos hold the buckets' entries, er / es the lists of epsilon arcs.
// (Its inputs are hidden from the compiler, so that it takes no registers from the light frame; see k_advance.)
template <int NT, bool TEAM>
__device__ __forceinline__ int heavy_frame(ConstDev *Dp, int my_lane, int chan) {
  using HC = HeavyCfg<NT>;
  asm volatile("" : "+s"(Dp), "+s"(my_lane), "+s"(chan));
  ConstDev &D = *(ConstDev *)uni((unsigned long long)Dp);
  LaneShared<NT> &S = lane_lds<NT, TEAM>();
  my_lane = uni(my_lane); chan = uni(chan);
  TeamCtx W = S.team;                               // (the same for every thread: in scalar registers)
  W.tl = D.teams + my_lane; W.g = uni(W.g); W.G = uni(W.G); W.spin_limit = uni(W.spin_limit);
  W.seq = uni(W.seq); W.pass = uni(W.pass); W.same_xcd = uni(W.same_xcd);
  Aux *const aux = D.aux + (size_t)my_lane * (size_t)D.auxcap;
  uint32_t *const infos = D.queue + (size_t)my_lane * (size_t)D.qcap;
  uint32_t *const er = D.dkey + (size_t)my_lane * (size_t)D.tokcap, *const es = D.dslot + (size_t)my_lane * (size_t)D.tokcap;
  long long *const foff = D.frame_off + (size_t)chan * (size_t)(D.max_frames + 2);
  HTok *const hist = D.hist + (size_t)chan * (size_t)D.hist_cap;
  LatInt *const lat = D.lat + (size_t)chan * (size_t)D.lat_cap;
  constexpr uint32_t mask = HC::SLOTS - 1;
  constexpr int hbits = HC::HBITS;
  constexpr int U = 4;
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int lane = tid & 63, wid = uni(tid >> 6);
  const unsigned long long below = (1ull << lane) - 1ull;
  const uint32_t G = TEAM ? (uint32_t)W.G : 1u, g = TEAM ? (uint32_t)W.g : 0u;
  auto &C = heavy_counters<NT, TEAM>(S, W);
  auto R32 = [&](const uint32_t *p) -> uint32_t { if constexpr (TEAM) return ld32(p); else return *p; };
  const bool lead = g == 0 && tid == 0;
  const uint32_t *rec = D.g.rec;
  HeavyState hs = S.hs;                             // (the same for every thread: in scalar registers)
  hs.ll = uni(hs.ll); hs.in_off = uni(hs.in_off); hs.hist_used = uni(hs.hist_used);
  hs.lat_pos = uni(hs.lat_pos); hs.lat_room = uni(hs.lat_room); hs.nf = uni(hs.nf); hs.n_in = uni(hs.n_in);
  Slot *slots = S.hv.table;
  HeavyLocal &H = S.hl;
  const float *ll = hs.ll;
  const int nf = hs.nf;
  const long long out_base = hs.hist_used;

  // capacities of a bucket, of a workgroup's list of epsilon arcs; the last entries of infos hold the selection's list
  const uint32_t n_all = (uint32_t)max(0, min(D.auxcap, D.qcap - 2 * HEAVY_LIST));
  const uint32_t cap = n_all / (G * G), ecap = (uint32_t)D.tokcap / G;
  unsigned long long *const sel_list = reinterpret_cast<unsigned long long *>(infos + ((D.qcap - 2 * HEAVY_LIST) & ~1));
  uint32_t *const my_er = er + (size_t)g * ecap, *const my_es = es + (size_t)g * ecap;
  auto bucket = [&](uint32_t owner, uint32_t sender) { return (size_t)(owner * G + sender) * cap; };
  auto owner_of = [&](uint32_t h) -> uint32_t {
    if constexpr (!TEAM) return 0u;
    return (((h * 0x85EBCA6Bu) >> 16) * G) >> 16;
  };
  uint32_t phase = 0;                               // barriers passed in this frame
  // What the workgroups tell each other at barrier k: event bits and the number of candidates sent,
  // in word k % 3 (zeroed one barrier ahead), so that all of them read the same value after it.
  auto given_up = [&]() -> int {                    // (by all workgroups, after the same barrier)
    if (tid == 0) { S.team.seq = W.seq + 1; S.team.pass = W.pass; }
    __syncthreads();
    return HEAVY_GIVEN_UP;
  };
  auto sync = [&]() -> bool {
    if (lead) C.ev[(phase + 1) % 3] = 0;
    if constexpr (TEAM) { if (!team_sync<NT>(W, S)) return false; } else __syncthreads();
    ++phase;
    return true;
  };
  auto events = [&]() -> uint32_t { return uni(R32(&C.ev[(phase - 1) % 3])); };   // of the barrier just passed
  auto tell = [&](uint32_t bits) { atomicOr(&C.ev[phase % 3], bits); };
#ifdef WFST_PHASE_TIMING
  if (threadIdx.x == 0) S.gtlast = wall_clock64();
#endif

  if constexpr (!TEAM) {
    if (tid == 0) reset_heavy(C);
  }
  if (tid == 0) {
    H.best = KEY_NONE; H.ctr = 0; H.again = 0; H.fail = 0; H.lat_full = 0; H.kept = 0; H.sent = 0;
  }
  if (tid < TEAM_MAX) { H.to[tid] = 0; H.upto[tid] = 0; }
  {                                                 // the LDS was the light frame's, or the last frame's
    const Slot fresh{~0ull, EMPTY, 0xFFFFFFFFu};
    for (int i = tid; i < HC::SLOTS; i += NT) slots[i] = fresh;
  }
  // touch this frame's row of scores, so that the gathers by pdf id below hit L2
  float touch = 0.f;
  for (int p = tid * 16; p < D.g.num_pdfs; p += NT * 16) touch += ll[p];

  // A candidate for another owner, or (one workgroup) for the table: into the owner's bucket.
  auto push = [&](bool want, uint32_t dw, float x, uint32_t arc, uint32_t src, uint32_t info) {
    if (!want) return;
    const uint32_t o = owner_of(dw & HMASK);
    uint32_t p;
    if constexpr (TEAM) p = atomicAdd(&H.to[o], 1u); else p = wave_alloc(&H.to[0]);
    if (p >= cap) { H.fail = 1; return; }
    const size_t at = bucket(o, g) + p;
    aux[at] = Aux{dw, x, arc, src};
    infos[at] = info;
  };
  auto publish = [&]() {                            // how far this workgroup's buckets are filled, for the next barrier
    __syncthreads();
    if (tid < (int)G) C.cnt[phase & 1][tid][g] = min(H.to[tid], cap);
    if (tid == 0 && H.fail) tell(EV_FAIL);
  };

  // ---- 1. emitting expansion ------------------------------------------------------------------
  unsigned long long emit_arcs = 0;
  {
    const long long in_off = hs.in_off;
    const int t0 = (int)((long long)hs.n_in * g / G), t1 = (int)((long long)hs.n_in * (g + 1) / G);
    for (int tb = t0; tb < t1; tb += NT) {
      uint32_t h = 0; float c = 0.f; int ne = 0;
      if (tb + tid < t1) {
        const HTok t = hist[in_off + tb + tid];
        h = t.handle & HMASK; c = t.cost;
        ne = (int)rec[3 * (size_t)h];
      }
      int total;
      const int ex = block_excl_scan<NT>(ne, S.wave_tmp, total);
      S.scan[tid] = ex; S.cost[tid] = c; S.base[tid] = h + 1;
      __syncthreads();
      GEN_MARK(8);
      total = uni(total);
      emit_arcs += (unsigned long long)total;
      // one thread per arc (Section 3.3), U arcs of the tile per thread and round so that their
      // loads are in flight together
      for (int j0 = 0; j0 < total; j0 += NT * U) {
        float x[U], ct[U], sll[U]; uint32_t r[U], dw[U], kx[U], wt[U], w2[U]; int kk[U];
        int lo[U], hi[U], jc[U];
#pragma unroll
        for (int u = 0; u < U; ++u) { jc[u] = min(j0 + u * NT + tid, total - 1); lo[u] = 0; hi[u] = NT - 1; }
        constexpr int STEPS = NT >= 1024 ? 10 : NT >= 512 ? 9 : 8;
#pragma unroll
        for (int it = 0; it < STEPS; ++it) {        // largest k with scan[k] <= j
          int v[U];
#pragma unroll
          for (int u = 0; u < U; ++u) v[u] = S.scan[(lo[u] + hi[u] + 1) >> 1];
#pragma unroll
          for (int u = 0; u < U; ++u) { const int mid = (lo[u] + hi[u] + 1) >> 1; if (v[u] <= jc[u]) lo[u] = mid; else hi[u] = mid - 1; }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
          kk[u] = tb + lo[u];
          r[u] = S.base[lo[u]] + (uint32_t)(jc[u] - S.scan[lo[u]]);
          ct[u] = S.cost[lo[u]];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const uint32_t *a = rec + 3 * (size_t)r[u];
          dw[u] = a[0]; wt[u] = a[1]; w2[u] = a[2];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < U; ++u) sll[u] = ll[w2[u] & D.g.pdf_mask];
        __builtin_amdgcn_sched_barrier(0);
        uint32_t m = KEY_NONE;
        int bad = 0;
#pragma unroll
        for (int u = 0; u < U; ++u) {
          x[u] = (ct[u] + __uint_as_float(wt[u])) - sll[u];
          const int have = (int)(j0 + u * NT + tid < total), fine = (int)(x[u] > -INFINITY);   // (neither NaN nor -inf)
          bad |= have & (fine ^ 1);
          kx[u] = (have & fine) ? okey(x[u]) : KEY_NONE;
          m = min(m, kx[u]);
        }
        if (bad) tell(EV_NAN);
        m = wave_min_u32(m);
        if (lane == 0 && m != KEY_NONE) atomicMin(&H.best, m);
        __syncthreads();
        const float cut = key2f(uni(H.best)) + D.beam;          // running bound, never below the final cutoff
#pragma unroll
        for (int u = 0; u < U; ++u)
          push(kx[u] != KEY_NONE && x[u] <= cut, dw[u], x[u], r[u], (uint32_t)kk[u], D.g.info_shift ? w2[u] >> 16 : INFO_UNKNOWN);
        GEN_MARK(9);
      }
      __syncthreads();
    }
  }
  asm volatile("" ::"v"(touch));
  publish();
  if (tid == 0) {
    if (H.best != KEY_NONE) atomicMin(&C.best, H.best);
    C.emit[g] = emit_arcs;
  }
  if (!sync()) return HEAVY_BROKEN;
  GEN_MARK(0);
  if constexpr (TEAM) { if (lead) reset_heavy(W.tl->ctr[(W.seq & 1) ^ 1]); }   // (the last frame's: everybody is past it)
  const uint32_t bestk = uni(R32(&C.best));
  uint32_t ev = events();
  if (ev & EV_FAIL) return given_up();
  int abort_code = 0;
  if (ev & EV_NAN) abort_code = E_NAN_INPUT;
  else if (bestk == KEY_NONE || bestk == KEY_PINF) abort_code = E_DEAD_CHANNEL;
  const float cutoff = key2f(bestk) + D.beam;

  // ---- 2 + 3. insertion and closure -----------------------------------------------------------
  // Offer a candidate to this workgroup's table; what the wave's lanes claimed or improved is
  // numbered and its epsilon arcs are listed, allotted once per wave.
  bool relaxing = false;                            // (before that an improved state's epsilon arcs are listed and not relaxed yet)
  auto offer = [&](bool want, uint32_t dw, float x, uint32_t arc, uint32_t info) {
    const uint32_t h = dw & HMASK;
    uint32_t sl = slot_hash(h, hbits), got = 0, tries = 0;
    bool is_new = false, again = false;
    if (want) {
      for (;;) {
        got = atomicCAS(&slots[sl].handle, EMPTY, h);
        if (got == EMPTY || got == h || ++tries >= HC::MAX_PROBES) break;
        sl = (sl + slot_step(h)) & mask;
      }
      if (got == EMPTY || got == h) {
        const unsigned long long old = atomicMin(&slots[sl].val, pack(okey(x), arc));
        is_new = got == EMPTY;
        again = !is_new && relaxing && (dw & HAS_EPS) && okey(x) < (uint32_t)(old >> 32);
      } else {
        H.fail = 1;
      }
    }
    const unsigned long long m_new = __ballot(is_new);
    if (!(m_new | __ballot(again))) return;
    uint32_t ne = info & INFO_NE, np = (info >> INFO_NP_SHIFT) & INFO_NP;
    const bool lists = (is_new || again) && (dw & HAS_EPS);
    if (lists && (ne == INFO_NE || np == INFO_NP)) { ne = rec[3 * (size_t)h]; np = rec[3 * (size_t)h + 1]; }
    const uint32_t v = lists ? min(np, 0xFFFFu) : 0u;
    const uint32_t inc = (uint32_t)wave_incl_scan((int)v);
    unsigned long long base = 0;
    if (lane == 63) base = atomicAdd(&H.ctr, ((unsigned long long)inc << 32) | (unsigned long long)__popcll(m_new));
    const uint32_t ci = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)base, 63) + (uint32_t)__popcll(m_new & below);
    const uint32_t e0 = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(base >> 32), 63) + inc - v;
    if (is_new) {
      if (ci >= (uint32_t)HC::CLAIM_LIMIT) H.fail = 1;
      else { S.hv.lq[ci] = (uint16_t)sl; slots[sl].aux = ((info & 0xFFFFu) << 16) | ci; }
    }
    if (lists) {
      if (np > 0xFFFFu || e0 + np > ecap) H.fail = 1;
      else {
        if (again) atomicAdd(&H.again, np);
        for (uint32_t k = 0; k < np; ++k) { my_er[e0 + k] = h + 1 + ne + k; my_es[e0 + k] = sl | (again ? EL_AGAIN : 0u); }
      }
    }
  };
  // The candidates that have arrived in this workgroup's buckets since it last looked: fn(mine, entry, info).
  auto arrivals = [&](uint32_t which, auto fn) {
    if (tid < (int)G) {
      const uint32_t n = R32(&C.cnt[which][g][tid]);
      H.from[tid] = H.upto[tid];
      H.upto[tid] = n;
    }
    __syncthreads();
    uint32_t total = 0;
    for (uint32_t s = 0; s < G; ++s) total += uni(H.upto[s]) - uni(H.from[s]);
#pragma unroll 1
    for (uint32_t j0 = wid * 64; j0 < total; j0 += NT) {
      uint32_t j = min(j0 + lane, total - 1), s = 0;
      if constexpr (TEAM) {                         // the sender it came from
        for (;;) { const uint32_t n = H.upto[s] - H.from[s]; if (j < n) break; j -= n; ++s; }
      }
      const size_t at = bucket(g, s) + H.from[s] + j;
      fn(j0 + lane < total, aux[at], infos[at]);
    }
  };
  int rounds = 0;
  uint32_t e_done = 0;                              // listed epsilon arcs relaxed so far
  if (abort_code == 0) {
    arrivals(0, [&](bool mine, const Aux &a, uint32_t info) { offer(mine && a.x <= cutoff, a.slot, a.x, a.arc, info); });
    if (tid < TEAM_MAX) H.emitted[tid] = H.upto[tid];           // (what comes later is not emitting)
    relaxing = true;
    GEN_MARK(10);
    for (;;) {
      for (;;) {                                    // this workgroup's own epsilon arcs, until none is left
        __syncthreads();
        const uint32_t e_end = min(uni((uint32_t)(H.ctr >> 32)), ecap);
        const bool stop = uni(H.fail) != 0;
        __syncthreads();
        if (e_done >= e_end || stop) break;
        ++rounds;
#pragma unroll 1
        for (uint32_t i0 = e_done + wid * 64; i0 < e_end; i0 += NT) {
          const uint32_t i = min(i0 + lane, e_end - 1);
          const uint32_t re = my_er[i], sl = my_es[i] & ~EL_AGAIN;
          const uint32_t *a = rec + 3 * (size_t)re;
          const uint32_t dw = a[0]; const float w = __uint_as_float(a[1]); const uint32_t w2 = a[2];
          const float xe = key2f(reinterpret_cast<const uint32_t *>(&slots[sl].val)[1]) + w;
          const bool want = i0 + lane < e_end && xe <= cutoff;
          const uint32_t info = D.g.info_shift ? w2 >> 16 : INFO_UNKNOWN;
          const bool here = !TEAM || owner_of(dw & HMASK) == g;
          if constexpr (TEAM) {
            push(want && !here, dw, xe, re, 0u, info);
            const unsigned long long m = __ballot(want && !here);
            if (m && lane == 0) atomicAdd(&H.sent, (uint32_t)__popcll(m));
          }
          offer(want && here, dw, xe, re, info);
        }
        e_done = e_end;
      }
      if constexpr (!TEAM) break;
      publish();
      if (tid == 0) {
        if (H.sent) atomicAdd(&C.ev[phase % 3], H.sent);
        H.sent = 0;
        C.claims[phase & 1][g] = (uint32_t)H.ctr;
      }
      if (!sync()) return HEAVY_BROKEN;
      GEN_MARK(11);
      ev = events();
      if (ev & EV_FAIL) return given_up();
      if ((ev & EV_COUNT) == 0) break;
      arrivals((phase - 1) & 1, [&](bool mine, const Aux &a, uint32_t info) { offer(mine && a.x <= cutoff, a.slot, a.x, a.arc, info); });
    }
    if constexpr (!TEAM) { if (uni(H.fail)) return given_up(); }
  }
  GEN_MARK(1);

  // ---- 4. max-active --------------------------------------------------------------------------
  const uint32_t my_claims = abort_code == 0 ? uni((uint32_t)H.ctr) : 0u;
  uint32_t nclaim = my_claims;
  if constexpr (TEAM) {
    if (abort_code == 0) {
      nclaim = 0;
      for (uint32_t s = 0; s < G; ++s) nclaim += uni(R32(&C.claims[(phase - 1) & 1][s]));
    }
  }
  if (nclaim > (uint32_t)D.tokcap) return given_up();           // (the general frame reports it)
  uint32_t n_valid = nclaim;
  const uint32_t room = (uint32_t)min((long long)0x7FFFFFFF, D.hist_cap - out_base);
  if (abort_code == 0 && (D.approximate ? nclaim : min(nclaim, (uint32_t)D.max_active)) > room) { abort_code = E_HISTORY_OVERFLOW; n_valid = 0; }
  // kept: (cost, state) at most theta, compared as one 64-bit number
  unsigned long long theta = ~0ull;
  float cutoff_eff = cutoff;
  auto pair_of = [&](int i) { const Slot *s = slots + S.hv.lq[i]; return ((s->val >> 32) << 32) | (unsigned long long)s->handle; };
  if (abort_code == 0 && nclaim > (uint32_t)D.max_active) {
    unsigned long long lo = (unsigned long long)bestk << 32, hi = ((unsigned long long)okey(cutoff) << 32) | 0xFFFFFFFFull;
    if (D.approximate) {                            // that histogram spans the costs there are
      uint32_t kmax = 0;
      for (int i = tid; i < (int)my_claims; i += NT) kmax = max(kmax, (uint32_t)(pair_of(i) >> 32));
      kmax = ~wave_min_u32(~kmax);
      if (lane == 0) atomicMax(&C.kmax, kmax);
      if (!sync()) return HEAVY_BROKEN;
      lo = bestk; hi = uni(R32(&C.kmax));           // (of the costs alone)
    }
    uint32_t need = (uint32_t)D.max_active;
    for (;;) {
      int shift = 0;
      while (((hi - lo) >> shift) >= (unsigned long long)NBINS) ++shift;
      for (int b = tid; b < NBINS; b += NT) S.hist[b] = 0;
      __syncthreads();
      for (int i = tid; i < (int)my_claims; i += NT) {
        const unsigned long long v = D.approximate ? pair_of(i) >> 32 : pair_of(i);
        if (v >= lo && v <= hi) atomicAdd(&S.hist[(uint32_t)((v - lo) >> shift)], 1u);
      }
      __syncthreads();
      constexpr int PER = NBINS / NT;
      uint32_t loc[PER], sum = 0;
      if constexpr (TEAM) {
        uint32_t *gh = W.tl->hist[W.pass % 3], *gh_next = W.tl->hist[(W.pass + 2) % 3];
        ++W.pass;
        for (int b = tid; b < NBINS; b += NT) { const uint32_t cnt = S.hist[b]; if (cnt) atomicAdd(&gh[b], cnt); }
        if (!sync()) return HEAVY_BROKEN;
#pragma unroll
        for (int q = 0; q < PER; ++q) { loc[q] = ld32(&gh[tid * PER + q]); sum += loc[q]; }
        for (uint32_t b = g * NT + tid; b < (uint32_t)NBINS; b += G * NT) gh_next[b] = 0;
      } else {
#pragma unroll
        for (int q = 0; q < PER; ++q) { loc[q] = S.hist[tid * PER + q]; sum += loc[q]; }
      }
      int total;
      uint32_t run = (uint32_t)block_excl_scan<NT>((int)sum, S.wave_tmp, total);
#pragma unroll
      for (int q = 0; q < PER; ++q) {
        if (run < need && run + loc[q] >= need) { S.sel_bin = tid * PER + q; S.sel_below = run; S.sel_cnt = loc[q]; }
        run += loc[q];
      }
      __syncthreads();
      const uint32_t b = uni(S.sel_bin), nbelow = uni(S.sel_below), cnt = uni(S.sel_cnt);
      __syncthreads();
      const unsigned long long edge = min(hi, lo + ((unsigned long long)(b + 1) << shift) - 1ull);
      if (D.approximate) { theta = (edge << 32) | 0xFFFFFFFFull; break; }          // the bin's upper edge
      need -= nbelow;
      lo += (unsigned long long)b << shift; hi = edge;
      if (lo == hi) { theta = lo; break; }
      if (cnt > (uint32_t)HEAVY_LIST) continue;
      // few enough to list them and rank each among all
      for (int i0 = wid * 64; i0 < (int)my_claims; i0 += NT) {
        const unsigned long long v = i0 + lane < (int)my_claims ? pair_of(i0 + lane) : ~0ull;
        const bool in = v >= lo && v <= hi;
        const unsigned long long m = __ballot(in);
        if (!m) continue;
        uint32_t p = 0;
        if (lane == 0) p = atomicAdd(&C.listed, (uint32_t)__popcll(m));
        p = uni(p) + (uint32_t)__popcll(m & below);
        if (in && p < (uint32_t)HEAVY_LIST) sel_list[p] = v;
      }
      if (!sync()) return HEAVY_BROKEN;
      {
        const uint32_t n = min(cnt, (uint32_t)HEAVY_LIST);
        unsigned long long *sl = reinterpret_cast<unsigned long long *>(S.hist);      // (HEAVY_LIST pairs fit the histogram's place)
        for (uint32_t i = tid; i < n; i += NT) sl[i] = sel_list[i];
        __syncthreads();
        for (uint32_t k = tid; k < n; k += NT) {    // (HEAVY_LIST pairs are more than a workgroup of 256 threads has)
          const unsigned long long v = sl[k];
          uint32_t rank = 0;
          for (uint32_t i = 0; i < n; ++i) rank += sl[i] < v ? 1u : 0u;
          if (rank + 1 == need) S.sel_theta = v;
        }
        __syncthreads();
        theta = uni(S.sel_theta);
      }
      break;
    }
    cutoff_eff = key2f((uint32_t)(theta >> 32));
  }
  GEN_MARK(2);

  // ---- 5 + 6. token numbers, history records, back-pointers, lattice records -------------------
  uint32_t pos0 = 0;                                // number of this workgroup's first kept token
  if (abort_code == 0) {
    uint32_t my_kept = my_claims;
    if (theta != ~0ull) {
      for (int i0 = wid * 64; i0 < (int)my_claims; i0 += NT) {
        const int i = min(i0 + lane, (int)my_claims - 1);
        const bool keep = i0 + lane < (int)my_claims && pair_of(i) <= theta;
        const unsigned long long m = __ballot(keep);
        uint32_t p = 0;
        if (lane == 0 && m) p = atomicAdd(&H.kept, (uint32_t)__popcll(m));
        p = uni(p) + (uint32_t)__popcll(m & below);
        if (i0 + lane < (int)my_claims) {
          Slot *s = slots + S.hv.lq[i];
          s->aux = (s->aux & 0xFFFF0000u) | (keep ? p : POS_NONE);
        }
      }
      __syncthreads();
      my_kept = uni(H.kept);
    }
    if (tid == 0) H.pos0 = atomicAdd(&C.nout, my_kept);
    __syncthreads();
    pos0 = uni(H.pos0);
    const long long lat_base = hs.lat_pos, lat_room = hs.lat_room;
    auto emit_lat = [&](bool wanted, uint32_t arc, float extra, uint32_t dst, uint32_t src) {
      const unsigned long long m = __ballot(wanted);
      if (!m) return;
      uint32_t p = 0;
      if (lane == 0) p = atomicAdd(&C.latn, (uint32_t)__popcll(m));
      p = uni(p) + (uint32_t)__popcll(m & below);
      if (!wanted) return;
      if ((long long)p >= lat_room) { H.lat_full = 1; return; }
      long long at = lat_base + (long long)p;
      if (at >= D.lat_cap) at -= D.lat_cap;
      lat[at] = LatInt{nf, arc, extra, dst, src};
    };
    // A candidate with its final cost: the one equal to the table's minimum is the token's best
    // incoming arc.  prev: as in the history record; NO_ARC if the source was cut by max-active (the
    // token is then left without a back-pointer and no lattice arc is recorded).
    auto settle = [&](bool mine, uint32_t h, float x, uint32_t arc, uint32_t prev) {
      bool wanted = false;
      float extra = 0.f;
      uint32_t dst = 0;
      if (mine && x <= cutoff_eff) {
        const int f = ht_find<true>(slots, mask, hbits, h);
        if (f >= 0) {
          const Slot sv = ld_slot<true>(slots + f);
          const uint32_t pos = sv.aux & POS_NONE;
          if (pos != POS_NONE) {
            dst = pos0 + pos;
            if (pack(okey(x), arc) == sv.val)
              hist[out_base + dst] = HTok{sv.handle | ((sv.aux >> (16 + INFO_NP_SHIFT)) ? HAS_EPS : 0u), x, arc, prev};
            extra = x - key2f((uint32_t)(sv.val >> 32));
            wanted = D.lattice_on && prev != NO_ARC && extra <= D.lattice_beam;
          }
        }
      }
      emit_lat(wanted, arc, extra, dst, prev);
    };
    // its own epsilon arcs first: what others own is on its way while the emitting candidates are settled
    const uint32_t e_end = min(uni((uint32_t)(H.ctr >> 32)), ecap);
    for (uint32_t i0 = wid * 64; i0 < e_end; i0 += NT) {
      const uint32_t i = min(i0 + lane, e_end - 1);
      const uint32_t re = my_er[i], esl = my_es[i];
      const uint32_t *a = rec + 3 * (size_t)re;
      const uint32_t dw = a[0]; const float w = __uint_as_float(a[1]);
      const Slot sv = ld_slot<true>(slots + (esl & ~EL_AGAIN));
      const float xe = key2f((uint32_t)(sv.val >> 32)) + w;
      const uint32_t spos = sv.aux & POS_NONE, prev = spos == POS_NONE ? NO_ARC : ((pos0 + spos) | PREV_SAME);
      const bool want = i0 + lane < e_end && !(esl & EL_AGAIN) && xe <= cutoff_eff;
      const bool here = !TEAM || owner_of(dw & HMASK) == g;
      if constexpr (TEAM) push(want && !here, dw, xe, re, prev, 0u);
      settle(want && here, dw & HMASK, xe, re, prev);
    }
    if constexpr (TEAM) publish();
    // the emitting candidates
    uint32_t total = 0;
    for (uint32_t s = 0; s < G; ++s) total += uni(H.emitted[s]);
#pragma unroll 1
    for (uint32_t j0 = wid * 64; j0 < total; j0 += NT) {
      uint32_t j = min(j0 + lane, total - 1), s = 0;
      if constexpr (TEAM) { for (;;) { const uint32_t n = H.emitted[s]; if (j < n) break; j -= n; ++s; } }
      const Aux a = aux[bucket(g, s) + j];
      settle(j0 + lane < total, a.slot & HMASK, a.x, a.arc, a.src);
    }
    if constexpr (TEAM) {
      if (!sync()) return HEAVY_BROKEN;
      ev = events();
      if (ev & EV_FAIL) abort_code = 1;             // (a bucket overflowed: nothing of the frame counts yet)
      else arrivals((phase - 1) & 1, [&](bool mine, const Aux &a, uint32_t) { settle(mine, a.slot & HMASK, a.x, a.arc, a.src); });
      if (abort_code == 1) return given_up();
    }
    __syncthreads();
    if (tid == 0) {
      if (H.lat_full) tell(EV_LATOVF);
      C.eps[g] = (uint32_t)(H.ctr >> 32) - H.again;
    }
  }
  if (!sync()) return HEAVY_BROKEN;
  GEN_MARK(3);
  if (g == 0 && tid == 0) {                         // the lane's state after the frame
    const uint32_t evd = R32(&C.ev[(phase - 1) % 3]);
    if (abort_code == 0 && (evd & EV_LATOVF)) abort_code = E_LATTICE_OVERFLOW;
    const uint32_t n_out = n_valid ? R32(&C.nout) : 0u;
    const long long lat_new = min((long long)(n_valid ? R32(&C.latn) : 0u), hs.lat_room);
    unsigned long long arcs = 0;
    for (uint32_t s = 0; s < G; ++s) {
      if constexpr (TEAM) arcs += ld64(&C.emit[s]); else arcs += C.emit[s];
      if (n_valid) arcs += R32(&C.eps[s]);
    }
    foff[nf + 1] = out_base + n_out;
    S.nf = nf + 1;
    S.in_off = out_base; S.n_in = (int)n_out;
    S.hist_used = out_base + n_out;
    S.lat_total += lat_new; S.lat_room -= lat_new;
    S.lat_pos += lat_new;
    if (S.lat_pos >= D.lat_cap) S.lat_pos -= D.lat_cap;
    S.arcs_expanded += (long long)arcs;
    S.max_pre = max(S.max_pre, (int)n_valid);
    S.max_post = max(S.max_post, (int)n_out);
    S.iters_max = max(S.iters_max, rounds);
#ifdef WFST_PHASE_TIMING
    S.ph[7] += rounds; S.dbg_tok += n_out;
#endif
    if (abort_code != 0) S.status = abort_code;
  }
  if (tid == 0) { S.team.seq = W.seq + 1; S.team.pass = W.pass; }
  __syncthreads();
  GEN_MARK(4);
  return HEAVY_DONE;
}

}  // namespace wfst
