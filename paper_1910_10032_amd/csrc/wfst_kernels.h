// Kernels of the decoder.
//
// One workgroup owns one lane (one audio stream of the batch) for a whole advance call and
// loops over that lane's frames by itself: streams are independent and frames are strictly
// serial (the paper's Section 3.1), so lanes never wait for each other and between the stages of
// a frame stand workgroup barriers.  This takes the paper's "one CTA per utterance" persistent
// kernel for the tail of the non-emitting iterations (Section 3.3) and applies it to the entire
// frame: with hundreds of lanes resident the chip is filled by lanes rather than by the arcs of
// one lane, and no kernel launch sits between the stages of Fig. 1.  A call of so few lanes that
// compute units would stand idle gives each lane further workgroups, a team, which share the
// frames of thousands of tokens with the first one, with barriers of the team in between.
//
// A frame takes the first of three forms that it fits: light (everything in the LDS of one
// workgroup, wfst_frame_light.h), heavy (state table in the LDS of one workgroup or of a team,
// wfst_frame_heavy.h), general (any size, table in memory, wfst_frame_general.h).  What a frame
// computes is the same in all of them (Section 3, first paragraph; Fig. 1):
//   1. emitting expansion, load-balanced over arcs (one thread per outgoing arc, Section
//      3.3): x = (cost + weight) - loglike[pdf], and the lane's best cost;
//   2. candidates within best + beam enter the lane's state table through a 64-bit atomic
//      minimum over (ordered cost bits, arc index); then the non-emitting closure: rounds over
//      the newly added / improved tokens until a round adds nothing;
//   3. max-active: if more than max_active tokens are within the beam, an exact histogram
//      selection over (cost, state) finds the cut; its cost is the frame's effective cutoff
//      (the adaptive beam);
//   4. the kept tokens are numbered in the channel's token history, and are what the next frame
//      expands from;
//   5. lattice preprocessing (Section 3.4): every candidate arc that reaches a kept token
//      within the effective cutoff and the lattice beam is recorded with its extra cost;
//      the arc equal to the table's minimum fixes the token's back-pointer;
//   6. the table is cleared.
// A call may cover many chunks of frames: at the boundaries the caller names, the lane seals
// a snapshot of its channel (and hands its lattice records over in the caller's form) and
// goes on, so that partial results can be read beside the decoding and no lane waits for a
// slower one (the role of the paper's second stream, Section 3, Fig. 1).
#pragma once
#include "wfst_frame_general.h"
#include "wfst_frame_heavy.h"
#include "wfst_frame_light.h"

namespace wfst {

// Frames without a heavy one after which the extra workgroups of a lane leave (and for how many
// frames past its last heavy one a channel gets them at the start of a call).  With 16 most teams are
// gone before a stream's first heavy frame; more than 64 holds compute units longer for less: 16 / 64 /
// 256 frames, 150 streams at beam 18 14.7 / 9.0 / 8.6 ms, 100 at beam 16.5 14.1 / 12.8 / 12.7 ms.
constexpr int TEAM_PATIENCE = 64;

// An extra workgroup of a lane joins the lane's team, works through the heavy frames the first
// workgroup calls it to, and leaves when told to.  Nothing depends on it being there: the team is
// whoever has joined when the first heavy frame comes, so a workgroup that the device has no room
// for yet finds the team closed when it starts, and leaves.
template <int NT>
__device__ __forceinline__ bool team_join(LaneShared<NT> &S, TeamLane *tl, uint32_t launch) {
  if (threadIdx.x == 0) {
    uint32_t xcc;
    asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(xcc));
    uint32_t spins = 0;
    while ((uint32_t)(ld64(&tl->join) >> 32) != launch && ++spins <= TEAM_SPIN_LIMIT) __builtin_amdgcn_s_sleep(2);   // the first workgroup sets the lane up
    S.team_cmd = 0;
    if (spins <= TEAM_SPIN_LIMIT) {
      const uint32_t before = atomicOr(&tl->xcc_mask, 1u << (xcc & 31u));
      asm volatile("" ::"v"(before));               // (the mask is complete before the count says so)
      const unsigned long long v = atomicAdd(&tl->join, 1ull);
      const uint32_t g = (uint32_t)(v & 0xFFFFu) + 1u;
      if (!(v & TEAM_CLOSED) && g < (uint32_t)TEAM_MAX) { S.team_cmd = 1; S.team.g = (int)g; }
    }
  }
  __syncthreads();
  return uni(S.team_cmd) != 0;
}
// Waits for the next command; false: leave.
template <int NT>
__device__ __forceinline__ bool team_next(LaneShared<NT> &S, TeamLane *tl) {
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t polls = 0;
    const uint32_t seen = S.team.commands;
    while (ld32(&tl->cmd_seq) == seen && !ld32(&tl->broken) && ++polls != 0xFFFFFFFFu) __builtin_amdgcn_s_sleep(2);
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    S.team_cmd = ld32(&tl->cmd_seq) == seen ? (uint32_t)TEAM_EXIT : ld32(&tl->cmd);
    S.hs = tl->hs;
    S.team.G = (int)tl->G; S.team.same_xcd = tl->same_xcd; S.team.commands = seen + 1u;
  }
  __syncthreads();
  return uni(S.team_cmd) == (uint32_t)TEAM_FRAME;
}

// One workgroup per lane, or (TEAM) several: the first n_lanes8 (the number of lanes, rounded up to
// a multiple of the eight XCDs) blocks are the lanes' first workgroups, the others join them, those
// of a lane on the same XCD.  is_init: (re)start the lane's channel and write frame 0.
// Between frames the lane's state is held in registers by every thread (LaneCtx, all values
// uniform); a general or heavy frame gets it through LDS.
// Readouts of snapshots run beside this kernel, on compute units that are full of lanes: of the 512
// vector registers of a SIMD lane the four wavefronts that a unit's lanes have there take 4 * 112 (the
// attribute counts pairs), and the readout kernels make do with the other 64.  For the same reason
// nothing here goes to scratch memory (while a kernel with scratch runs, kernels of another
// queue did not start before its first workgroups ended: 500 online streams got the first of 16
// partial results after 8.7 of 11.4 ms; now after 1.3 of 10.9).  Two things hold both: the three forms of
// a frame are inlined, and each takes the thread number and the decoder's description anew
// (asm volatile), so that nothing derived from them is computed before the frame loop and kept.
template <int NT, bool TEAM>
__global__ void __launch_bounds__(NT, NT >= 512 ? 4 : 2) __attribute__((amdgpu_num_vgpr(56))) k_advance(DecDev D, const DecDev *Dg, const LaneParam *__restrict__ lanes, int is_init, int n_lanes, int n_lanes8,
                                                                   uint32_t launch) {
  LaneShared<NT> &S = lane_lds<NT, TEAM>();
  const int tid = threadIdx.x;
  const bool member = TEAM && (int)blockIdx.x >= n_lanes8;          // an extra workgroup of a lane
  int my_lane = uni(member ? ((int)blockIdx.x - n_lanes8) % n_lanes8 : (int)blockIdx.x);
  if (TEAM && my_lane >= n_lanes) return;
  TeamLane *const tl = D.teams + my_lane;
  if (tid == 0) S.team = TeamCtx{tl, 0, 1, 0u, D.team_spin_limit, 0u, 0u, 0u, 0u};
  if (TEAM && member && !team_join<NT>(S, tl, launch)) return;
  asm volatile("" : "+s"(my_lane));                  // (the branch above meets here: without this what follows would be taken to depend on the thread)
  LaneParam lp = lanes[my_lane];
  lp.ll = uni(lp.ll); lp.chan = uni(lp.chan); lp.n_frames = uni(lp.n_frames); lp.stride = uni(lp.stride);
  lp.snap_every = uni(lp.snap_every); lp.snap_id0 = uni(lp.snap_id0); lp.n_snaps = uni(lp.n_snaps);
  ChanState *cs = D.chan + lp.chan;
  long long *foff = D.frame_off + (size_t)lp.chan * (size_t)(D.max_frames + 2);
  LatInt *lat = D.lat + (size_t)lp.chan * (size_t)D.lat_cap;

  const Slot fresh{~0ull, EMPTY, 0xFFFFFFFFu};
  for (int i = tid; i < LightCfg<NT>::SLOTS; i += NT) S.table[i] = fresh;
  constexpr int MW = LightCfg<NT>::MARK_WORDS;
  for (int i = tid; i < 2 * MW; i += NT) S.mark[i / MW][i % MW] = make_uint2(0, 0);
  if (tid == 0) {
    reset_ctr(S.fc[0]); reset_ctr(S.fc[1]);
    if (is_init) foff[0] = 0;
#ifdef WFST_PHASE_TIMING
    for (int k = 0; k < 16; ++k) { S.ph[k] = 0; S.gph[k] = 0; }
    S.dbg_tok = 0; S.dbg_iters = 0; S.dbg_arcs = 0;
#endif
  }
  LaneCtx ctx;
#ifdef WFST_PHASE_TIMING
  ctx.tlast = wall_clock64();
#endif
  if (is_init) {
    ctx.status = 0; ctx.nf = 0; ctx.hist_used = 0; ctx.lat_pend = 0; ctx.lat_pos = 0; ctx.lat_total = 0;
    if (tid == 0) { S.arcs_expanded = 0; S.max_pre = 0; S.max_post = 0; S.iters_max = 0; }
  } else {
    ctx.status = uni(cs->status); ctx.nf = uni(cs->num_frames); ctx.hist_used = uni(cs->hist_used);
    ctx.lat_total = uni(cs->lat_total);
    ctx.lat_pend = ctx.lat_total - uni(cs->lat_head);
    ctx.lat_pos = ctx.lat_total % D.lat_cap;
    if (tid == 0) { S.arcs_expanded = cs->arcs_expanded; S.max_pre = cs->max_pre; S.max_post = cs->max_post; S.iters_max = cs->closure_iters_max; }
  }
  ctx.n_in = 0;
  if (!is_init && ctx.nf >= 1 && ctx.nf <= D.max_frames + 1) ctx.n_in = (int)(uni(foff[ctx.nf]) - uni(foff[ctx.nf - 1]));
  ctx.pending_clear = 0; ctx.par = 0; ctx.tok_valid = false; ctx.n_arcs = 0; ctx.n_dead = 0; ctx.lds_foreign = false;
  int last_heavy = is_init ? 0 : uni(cs->last_heavy);
  int n_heavy = 0, gave_up = 0x7FFFFFFF;             // frames that were not light; tokens of the last frame whose heavy form was given up
  // the lane's team: set up, and open to whoever is to join
  bool team_open = false, team_here = false;        // joining is possible; there are members to call
  if (TEAM && !member) {
    for (int i = tid; i < 3 * NBINS; i += NT) tl->hist[i / NBINS][i % NBINS] = 0;
    if (tid == 0) {
      uint32_t xcc;
      asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(xcc));
      tl->xcc_mask = 1u << (xcc & 31u);
      tl->cmd_seq = 0; tl->cmd = 0; tl->arrived = 0; tl->broken = 0;
      reset_heavy(tl->ctr[0]); reset_heavy(tl->ctr[1]);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (tid == 0) {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
      atomicExch(&tl->join, (unsigned long long)launch << 32);
    }
    team_open = true;
  }
  // (thread 0) nobody joins from here on; how many have
  auto team_close = [&]() -> uint32_t { return (uint32_t)(atomicOr(&tl->join, TEAM_CLOSED) & 0xFFFFu); };
  auto team_dismiss = [&]() {
    if constexpr (TEAM) {
      if (tid == 0) {
        if (team_open) (void)team_close();
        tl->cmd = TEAM_EXIT;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        atomicAdd(&tl->cmd_seq, 1u);
      }
      if (tid == 0) S.team.G = 1;                     // (read again after the next barriers only)
      team_open = false; team_here = false;
    }
  };
  __syncthreads();
  // Seal the lane's state as the next snapshot of this call.  With snapshot blocks the lattice
  // records not handed out yet move into the snapshot's block, in the caller's form (the lane
  // reserves its range with one compare-and-swap; the ring is empty afterwards).  Then
  // everything the workgroup has written is made visible to the whole system, then the
  // snapshot entry and the lane's progress word.  Readouts of the snapshot start only after
  // the host has seen the progress words of all lanes, so nothing ever waits inside a kernel.
  int n_sealed = 0;
  auto seal = [&]() {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the lattice records of the frames so far are where they are read below
    __syncthreads();
    const long long id = lp.snap_id0 + n_sealed;
    long long blk_start = 0, blk_count = 0;
    if (D.n_blk > 0 && D.lattice_on) {
      const int slot = (int)(id % D.n_blk);
      const long long n = ctx.lat_pend;
      if (tid == 0) {
        unsigned long long *used = &D.blk[slot].used;
        unsigned long long old = ld64(used);
        long long pos = -1;
        while ((long long)old + n <= D.blk_cap) {     // every failed swap means another lane got its range
          const unsigned long long seen = atomicCAS(used, old, old + (unsigned long long)n);
          if (seen == old) { pos = (long long)old; break; }
          old = seen;
        }
        S.blk_pos = pos;
      }
      __syncthreads();
      const long long pos = uni(S.blk_pos);
      if (pos < 0 && ctx.status == 0) ctx.status = E_LATTICE_OVERFLOW;
      if (pos >= 0) {
        LatRec *out = D.blk_recs + (size_t)slot * (size_t)D.blk_cap + (size_t)pos;
        const long long first = ctx.lat_pos >= n ? ctx.lat_pos - n : ctx.lat_pos - n + D.lat_cap;
        int mine = tid;
        asm volatile("" : "+v"(mine));                  // (computed here, not held in registers from the kernel's start)
        constexpr int U = 4;                            // records per thread in flight: the arc-id gathers are HBM round trips
        for (long long i0 = mine; i0 < n; i0 += (long long)NT * U) {
          LatInt r[U];
          uint32_t arc_id[U];
          // loads are unconditional (a lane past the end re-reads the last record) so that all of a
          // round's loads, and then all its gathers, are in flight together
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const long long i = min(i0 + (long long)u * NT, n - 1);
            r[u] = lat[first + i < D.lat_cap ? first + i : first + i - D.lat_cap];
          }
#pragma unroll
          for (int u = 0; u < U; ++u) arc_id[u] = D.g.orig[r[u].arc];
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const long long i = i0 + (long long)u * NT;
            if (i < n) out[i] = LatRec{r[u].frame, arc_id[u], r[u].extra};
          }
        }
        blk_start = pos; blk_count = n;
      }
      ctx.lat_pend = 0;
    }
    // Every thread's stores (tokens, lattice records, the block) must have reached the L2 before
    // thread 0 publishes: each wave waits until its own stores have been acknowledged, then the
    // barrier, then thread 0's system-scope release, which writes the L2's dirty lines back.
    // (One release per lane and snapshot: a device-scope fence in every thread would flush and
    // invalidate the cache eight times over and slows all lanes of the chip down noticeably.)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (tid == 0) {
      ChanSnap *sp = D.snap + (size_t)lp.chan * SNAP_RING + (size_t)(id % SNAP_RING);
      sp->lat_total = ctx.lat_total; sp->hist_used = ctx.hist_used; sp->status = ctx.status; sp->num_frames = ctx.nf;
      sp->blk_start = blk_start; sp->blk_count = blk_count;
      sp->id = id;
      __hip_atomic_store(D.lane_sealed + blockIdx.x, id, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
    }
    ++n_sealed;
  };
  // a frame in the general or heavy form: the lane's state goes through LDS
  // (every wave waits until its stores have been acknowledged: the history records of the light frame
  // before are read by the other workgroups of the lane's team as soon as they are called)
  auto state_to_lds = [&]() {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if (tid == 0) {
      S.status = ctx.status; S.nf = ctx.nf; S.n_in = ctx.n_in; S.in_off = ctx.hist_used - ctx.n_in; S.hist_used = ctx.hist_used;
      S.lat_room = D.lat_cap - ctx.lat_pend; S.lat_total = ctx.lat_total; S.lat_pos = ctx.lat_pos;
    }
    __syncthreads();
  };
  auto state_from_lds = [&]() {
    ctx.status = uni(S.status); ctx.nf = uni(S.nf); ctx.n_in = uni(S.n_in); ctx.hist_used = uni(S.hist_used);
    ctx.lat_pend = D.lat_cap - uni(S.lat_room); ctx.lat_total = uni(S.lat_total); ctx.lat_pos = uni(S.lat_pos);
    ctx.tok_valid = false;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (the frame's history records, which the next frame starts from)
    __syncthreads();                                  // all have read the state before the next such frame rewrites it
  };
  auto run_general = [&](const float *ll) {
    state_to_lds();
    general_frame<NT, TEAM>((ConstDev *)Dg, my_lane, lp.chan, ll, is_init);
    state_from_lds();
  };
  // a frame in the heavy form: what the first workgroup does before it
  auto call_team = [&](const float *ll) {
    state_to_lds();
    if (tid == 0) S.hs = HeavyState{ll, ctx.hist_used - ctx.n_in, ctx.hist_used, ctx.lat_pos, D.lat_cap - ctx.lat_pend, ctx.nf, ctx.n_in};
    ctx.lds_foreign = true; ctx.tok_valid = false; ctx.pending_clear = 0;
    if constexpr (TEAM) {
      if (team_open) {                                // the first heavy frame: the team is whoever has joined
        if (tid == 0) {
          const uint32_t want = (gridDim.x - 1u - (uint32_t)my_lane) / (uint32_t)n_lanes8;
          for (uint32_t polls = 0; polls < 64u && (uint32_t)(ld64(&tl->join) & 0xFFFFu) < want; ++polls) __builtin_amdgcn_s_sleep(4);
          const uint32_t joined = team_close();
          const uint32_t xccs = ld32(&tl->xcc_mask);
          S.team.G = (int)joined + 1; S.team.same_xcd = (xccs & (xccs - 1u)) == 0u;
          tl->G = joined + 1u; tl->same_xcd = S.team.same_xcd;
        }
        __syncthreads();
        team_open = false; team_here = uni(S.team.G) > 1;
      }
      __syncthreads();
      if (team_here && tid == 0) {
        tl->hs = S.hs;
        tl->cmd = TEAM_FRAME;
        if (S.team.same_xcd) asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); else __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        atomicAdd(&tl->cmd_seq, 1u);
      }
    }
    __syncthreads();
  };
  const int nframes = is_init ? 1 : lp.n_frames;
  const int n_snaps = is_init ? 0 : lp.n_snaps;
  const bool light_ok = D.g.info_shift != 0 && D.force_general == 0, heavy_ok = is_init == 0 && D.force_general == 0;
  if (TEAM && ctx.nf - last_heavy > TEAM_PATIENCE) team_dismiss();
  int until_seal = (!is_init && lp.snap_every > 0) ? lp.snap_every : 0x7FFFFFFF;
  for (int f = 0;;) {
    const bool more = member || (f < nframes && ctx.status == 0);
    if (more) {
      const float *ll = nullptr, *ll_next = nullptr;
      bool done = false, heavy = false;
      if (member) {
        if constexpr (TEAM) { if (!team_next<NT>(S, tl)) return; }
        heavy = true;
      } else {
        ll = is_init ? nullptr : lp.ll + (size_t)f * (size_t)lp.stride;
        ll_next = (!is_init && f + 1 < nframes) ? ll + lp.stride : nullptr;
        if (light_ok && (is_init || ctx.n_in <= LightCfg<NT>::CLAIM_LIMIT))
          done = light_frame<NT>(D, S, ctx, ll, ll_next, is_init != 0, lp.chan);
        if (done) {
          if (TEAM && (team_open || team_here) && ctx.nf - last_heavy > TEAM_PATIENCE) team_dismiss();
        } else {
#ifdef WFST_PHASE_TIMING
          if (tid == 0) S.ph[6] += 1;
#endif
          last_heavy = ctx.nf;
          ++n_heavy;
          // (a frame that starts from nearly as many tokens as one that did not fit will not fit either)
          heavy = heavy_ok && (long long)ctx.n_in * 8 < (long long)gave_up * 7;
          if (heavy) call_team(ll);
        }
      }
      if (heavy) {
        const int r = uni(heavy_frame<NT, TEAM>((ConstDev *)Dg, my_lane, lp.chan));
        if (member) {
          if (r == HEAVY_BROKEN) return;
          continue;
        }
        if (r == HEAVY_BROKEN) {                      // (what the team has written is incomplete: the channel stops)
          __syncthreads();
          if (tid == 0) S.status = E_DEVICE;
          __syncthreads();
        }
        done = r != HEAVY_GIVEN_UP;
        gave_up = done ? 0x7FFFFFFF : ctx.n_in;
        if (done) state_from_lds();
        PHASE_MARK(11);
      }
      if (!done) {
        run_general(ll);
        PHASE_MARK(10);
      }
#ifdef WFST_PHASE_TIMING
      if (tid == 0) S.ph[5] += 1;
#endif
      ++f;
      if (--until_seal != 0) continue;
      until_seal = lp.snap_every;
    }
    // a snapshot boundary - or the lane has run out of frames or stopped: it seals the
    // snapshots still due in the state it is in
    if (n_sealed >= n_snaps) { if (more) continue; break; }
    seal();
    PHASE_MARK(12);
  }
  if (TEAM && (team_open || team_here)) team_dismiss();
  __syncthreads();
  if (tid == 0) {
    cs->last_heavy = last_heavy;
    if (!is_init) D.lane_heavy[my_lane] = n_heavy;
    cs->status = ctx.status; cs->num_frames = ctx.nf; cs->hist_used = ctx.hist_used;
    cs->lat_total = ctx.lat_total; cs->arcs_expanded = S.arcs_expanded; cs->max_pre = S.max_pre;
    cs->max_post = S.max_post; cs->closure_iters_max = S.iters_max;
    if (is_init) cs->path_nf = 0;
    cs->lat_head = ctx.lat_total - ctx.lat_pend;
#ifdef WFST_PHASE_TIMING
    if (D.dbg) {
      for (int k = 0; k < 16; ++k) { atomicAdd(D.dbg + k, S.ph[k]); atomicAdd(D.dbg + 16 + 10240 + k, S.gph[k]); }
      unsigned long long tot = 0;
      for (int k = 0; k < 16; ++k) if (k != 5 && k != 6 && k != 7 && k != 13) tot += S.ph[k];
      D.dbg[16 + blockIdx.x] = tot;                     // this lane's time for the call
      D.dbg[16 + 2048 + blockIdx.x] = S.dbg_tok;
      D.dbg[16 + 4096 + blockIdx.x] = S.dbg_arcs;
      D.dbg[16 + 6144 + blockIdx.x] = S.ph[6];            // frames in the general form
      D.dbg[16 + 8192 + blockIdx.x] = S.ph[11];           // time in them
    }
#endif
  }
}

__global__ void k_fill_slots(Slot *slots, size_t n) {
  const Slot fresh{~0ull, EMPTY, A_FRESH};
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) slots[i] = fresh;
}

// ---- readouts ----------------------------------------------------------------------------
struct PathOut { int32_t status, n_words, n_arcs, reached_final; float total_cost; int32_t pad; long long word_off; };

// Arg-min over the last frame of a channel by the whole wave: packed (ordered cost, handle)
// minimum over all tokens and, if asked for, over tokens in final states (cost + final cost).
// Returns false if the channel has an error or no token; lane 0 gets the start of the walk.
// The channel's state as the readouts see it: live, or as sealed in snapshot `snap_id` (> 0).
struct ChanView { int status, num_frames; long long hist_used, lat_total; };
__device__ __forceinline__ ChanView chan_view(const DecDev &D, int ch, long long snap_id) {
  if (snap_id <= 0) {
    const ChanState *cs = D.chan + ch;
    return ChanView{cs->status, cs->num_frames, cs->hist_used, cs->lat_total};
  }
  const ChanSnap *sp = D.snap + (size_t)ch * SNAP_RING + (size_t)(snap_id % SNAP_RING);
  if (sp->id != snap_id) return ChanView{E_NOT_INIT, 0, 0, 0};     // the channel has no such snapshot (any more)
  return ChanView{sp->status, sp->num_frames, sp->hist_used, sp->lat_total};
}

__device__ __forceinline__ bool path_start(const DecDev &D, int ch, int use_final, const ChanView &cv, PathOut &po, int &F, int &cur) {
  const int lane = threadIdx.x;
  const long long *foff = D.frame_off + (size_t)ch * (size_t)(D.max_frames + 2);
  const HTok *hist = D.hist + (size_t)ch * (size_t)D.hist_cap;
  const uint32_t *rec = D.g.rec;
  if (cv.status != 0) { po.status = cv.status; return false; }
  F = cv.num_frames - 1;
  if (F < 0) { po.status = E_NOT_INIT; return false; }
  const long long o = foff[F];
  const int n = (int)(foff[F + 1] - o);
  unsigned long long bf = ~0ull, bn = ~0ull; int bfi = -1, bni = -1;
  constexpr int PU = 4;                        // tokens in flight (a lane past the end looks at the last one again)
  for (int i0 = lane; i0 < n; i0 += 64 * PU) {
    HTok t[PU]; float fc[PU];
#pragma unroll
    for (int u = 0; u < PU; ++u) t[u] = hist[o + min(i0 + u * 64, n - 1)];
#pragma unroll
    for (int u = 0; u < PU; ++u) fc[u] = use_final ? __uint_as_float(rec[3 * (size_t)(t[u].handle & HMASK) + 2]) : INFINITY;
#pragma unroll
    for (int u = 0; u < PU; ++u) {
      const uint32_t h = t[u].handle & HMASK;
      const int i = min(i0 + u * 64, n - 1);
      const unsigned long long kn = pack(okey(t[u].cost), h);
      if (kn < bn) { bn = kn; bni = i; }
      if (fc[u] != INFINITY) {
        const unsigned long long kf = pack(okey(t[u].cost + fc[u]), h);
        if (kf < bf) { bf = kf; bfi = i; }
      }
    }
  }
  for (int d = 32; d; d >>= 1) {
    unsigned long long o2 = __shfl_xor(bn, d, 64); int i2 = __shfl_xor(bni, d, 64);
    if (o2 < bn) { bn = o2; bni = i2; }
    o2 = __shfl_xor(bf, d, 64); i2 = __shfl_xor(bfi, d, 64);
    if (o2 < bf) { bf = o2; bfi = i2; }
  }
  if (n == 0) { po.status = E_DEAD_CHANNEL; return false; }
  if (use_final && bfi >= 0) { cur = bfi; po.total_cost = key2f((uint32_t)(bf >> 32)); po.reached_final = 1; }
  else { cur = bni; po.total_cost = key2f((uint32_t)(bn >> 32)); }
  return true;
}

// Best path of one channel with its arcs (one wave; lane 0 follows the back-pointers over the
// whole utterance).  Words / arcs are written right-aligned into cap-sized regions, so a
// single backward walk leaves them in path order.
__global__ void __launch_bounds__(64) k_best_path(DecDev D, const int32_t *chans, int use_final, long long snap_id,
                                                  int32_t *words, int words_cap, uint32_t *arcs, int arcs_cap,
                                                  PathOut *out) {
  const int ch = chans[blockIdx.x];
  const long long *foff = D.frame_off + (size_t)ch * (size_t)(D.max_frames + 2);
  const HTok *hist = D.hist + (size_t)ch * (size_t)D.hist_cap;
  PathOut po{0, 0, 0, 0, 0.f, 0, 0};
  int F = 0, cur = 0;
  const ChanView cv = chan_view(D, ch, snap_id);
  const bool ok = path_start(D, ch, use_final, cv, po, F, cur);
  if (threadIdx.x != 0) return;
  if (!ok) { out[blockIdx.x] = po; return; }
  int32_t *wout = words ? words + (size_t)blockIdx.x * words_cap : nullptr;
  uint32_t *aout = arcs ? arcs + (size_t)blockIdx.x * arcs_cap : nullptr;
  int f = F, nw = 0, na = 0;
  const long long max_steps = cv.hist_used + 1;
  for (long long step = 0;; ++step) {
    if (cur < 0 || (long long)cur >= foff[f + 1] - foff[f]) { po.status = E_BROKEN_TRACE; break; }
    const HTok t = hist[foff[f] + cur];
    if (t.in_arc == NO_ARC) break;
    if (t.prev == NO_ARC || step > max_steps) { po.status = E_BROKEN_TRACE; break; }
    if (aout && na < arcs_cap) aout[arcs_cap - 1 - na] = D.g.orig[t.in_arc];
    ++na;
    const int32_t w = D.g.label[t.in_arc];
    if (w != 0) { if (wout && nw < words_cap) wout[words_cap - 1 - nw] = w; ++nw; }
    if (t.prev & PREV_SAME) cur = (int)(t.prev & ~PREV_SAME);
    else { cur = (int)t.prev; --f; if (f < 0) { po.status = E_BROKEN_TRACE; break; } }
  }
  po.n_words = nw; po.n_arcs = na;
  if (po.status == 0 && ((wout && nw > words_cap) || (aout && na > arcs_cap))) po.status = E_CAPACITY;
  out[blockIdx.x] = po;
}

// Best-path words of many channels, one wave each.  Back-pointers are unique, so two best
// paths that share a token share everything before it: each channel remembers, per frame,
// the token through which its last traced path entered the frame and the words up to there;
// a new trace walks back only until it meets the remembered path (a chunk of frames plus the
// distance to the merge point, not the whole utterance) and splices the remembered prefix.
// The walk is a serial chain with one memory round trip per arc: where the frames start and what
// the remembered path entered them through is fetched a frame ahead.  (Fetched when needed, they
// made two more round trips per frame; 500 channels beside a decode kernel: 0.70 ms per readout.)
// Words go to words + po.word_off: gi * words_cap, or, if words_used is given, packed (allotted
// with one atomic add).
// One wave per channel, of at most 64 registers: what the lanes of a running decode kernel leave
// free on every compute unit (see k_advance).
__global__ void __launch_bounds__(64, 8) k_best_path_words(DecDev D, const int32_t *chans, int use_final, long long snap_id,
                                                        int32_t *words, int words_cap, unsigned long long *words_used, PathOut *out) {
  const int gi = blockIdx.x, ch = chans[gi], lane = threadIdx.x;
  ChanState *cs = D.chan + ch;
  const long long *foff = D.frame_off + (size_t)ch * (size_t)(D.max_frames + 2);
  const HTok *hist = D.hist + (size_t)ch * (size_t)D.hist_cap;
  int32_t *entry = D.pc_entry + (size_t)ch * (size_t)(D.max_frames + 2);
  int32_t *wcount = D.pc_wcount + (size_t)ch * (size_t)(D.max_frames + 2);
  int32_t *cw = D.pc_words + (size_t)ch * (size_t)D.pc_wcap;
  PathOut po{0, 0, 0, 0, 0.f, 0, 0};
  int F = 0, cur = 0;
  const ChanView cv = chan_view(D, ch, snap_id);
  const bool ok = path_start(D, ch, use_final, cv, po, F, cur);
  if (!ok) { if (lane == 0) out[gi] = po; return; }
  int status = 0, total = 0, merge_f = 0, k = 0;
  if (lane == 0) {
    const int cached_nf = cs->path_nf;
    int f = F, base = 0;
    const long long max_steps = cv.hist_used + 1;
    // start of frame f and of the next one, and, on their way, those of the frames before; the
    // remembered path's token in frame f, and in the frame before
    long long o = foff[f], o_end = foff[f + 1], o1 = f >= 1 ? foff[f - 1] : 0, o2 = f >= 2 ? foff[f - 2] : 0;
    auto remembered = [&](int ff) { return ff >= 0 && ff < cached_nf ? entry[ff] : -1; };
    int e0 = remembered(f), e1 = remembered(f - 1);
    HTok t{};
    if (cur < 0 || (long long)cur >= o_end - o) status = E_BROKEN_TRACE; else t = hist[o + cur];
    for (long long step = 0; status == 0; ++step) {
      if (t.in_arc == NO_ARC) break;
      if (t.prev == NO_ARC || step > max_steps) { status = E_BROKEN_TRACE; break; }
      const bool is_entry = !(t.prev & PREV_SAME);
      if (is_entry) {
        if (e0 >= 0 && e0 == cur) { base = wcount[f]; merge_f = f; break; }
        entry[f] = cur; wcount[f] = k;        // k: words found so far, all later on the path; fixed up below
        --f; o_end = o; o = o1; o1 = o2; o2 = f >= 2 ? foff[f - 2] : 0;
        e0 = e1; e1 = remembered(f - 1);
      }
      // the next token and this arc's word are fetched together
      cur = (int)(t.prev & ~PREV_SAME);
      const uint32_t arc = t.in_arc;
      const bool ok2 = f >= 0 && (long long)cur < o_end - o;
      if (ok2) t = hist[o + cur];
      const int32_t w = D.g.label[arc];
      if (w != 0) {
        if (k < D.pc_wcap) cw[D.pc_wcap - 1 - k] = w;
        ++k;
      }
      if (!ok2) status = E_BROKEN_TRACE;
    }
    if (status == 0 && (long long)base + 2ll * k > (long long)D.pc_wcap) status = E_CAPACITY;
    total = base + k;
  }
  status = uni(status); total = uni(total); merge_f = uni(merge_f); k = uni(k);
  __threadfence_block();                       // (the first lane's stores, before the others read them)
  if (status != 0) {
    if (lane == 0) { cs->path_nf = 0; po.status = status; po.n_words = total; out[gi] = po; }
    return;
  }
  for (int f = merge_f + 1 + lane; f <= F; f += 64) wcount[f] = total - wcount[f];
  const int base = total - k;
  for (int j = lane; j < k; j += 64) cw[base + j] = cw[D.pc_wcap - k + j];
  __threadfence_block();
  long long off = (long long)gi * words_cap;
  if (lane == 0) {
    cs->path_nf = F + 1;
    po.n_words = total;
    if (total > words_cap) po.status = E_CAPACITY;
    else if (words_used) off = (long long)atomicAdd(words_used, (unsigned long long)total);
    po.word_off = off;
    out[gi] = po;
  }
  po.status = uni(po.status);
  off = uni(off);
  if (po.status != 0) return;
  for (int j = lane; j < total; j += 64) words[off + j] = cw[j];
}

// Tokens of one frame in the public form: state id and caller's arc id.
struct TokOut { int32_t state; float cost; uint32_t in_arc; };
__global__ void k_export_tokens(DecDev D, int ch, long long off, int n, TokOut *out) {
  const HTok *hist = D.hist + (size_t)ch * (size_t)D.hist_cap;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    const HTok t = hist[off + i];
    out[i] = TokOut{D.g.label[t.handle & HMASK], t.cost, t.in_arc == NO_ARC ? NO_ARC : D.g.orig[t.in_arc]};
  }
}

// Lattice records with frame >= from_frame, arc ids translated to the caller's; cnt is
// the running output count (zeroed by the host).
// (the n records start at ring position `start`)
__global__ void k_export_lattice(DecDev D, int ch, long long start, long long n, int from_frame, LatRec *out, long long cap,
                                 unsigned long long *cnt) {
  const LatInt *lat = D.lat + (size_t)ch * (size_t)D.lat_cap;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x) {
    const LatInt r = lat[start + i < D.lat_cap ? start + i : start + i - D.lat_cap];
    if (r.frame < from_frame) continue;
    const unsigned long long p = atomicAdd(cnt, 1ull);
    if ((long long)p < cap) out[p] = LatRec{r.frame, D.g.orig[r.arc], r.extra};
  }
}
// Records a live drain hands out.  A channel stopped by an overflow hands out nothing.
__device__ __forceinline__ long long lattice_pending(const DecDev &D, int ch) {
  const ChanState *cs = D.chan + ch;
  const bool readable = cs->status == 0 || cs->status == E_DEAD_CHANNEL || cs->status == E_NAN_INPUT;
  return readable ? cs->lat_total - cs->lat_head : 0;
}
__global__ void k_reset_lattice(DecDev D, int ch) { D.chan[ch].lat_head = D.chan[ch].lat_total; }

// Batched drain: counts of the listed channels, then one copy kernel (grid.x = channel,
// grid.y = slices of that channel's buffer), then the reset.
// offs[0..n]: exclusive prefix sums of the buffered record counts of the listed channels
// (channels stopped by an overflow count as empty), also written to pinned host memory.  One block.
__global__ void __launch_bounds__(1024) k_lattice_offsets(DecDev D, const int32_t *chans, int n, long long *offs, long long *offs_host) {
  __shared__ long long part[1024];
  const int tid = threadIdx.x;
  const int per = (n + 1023) / 1024;
  const int b = tid * per, e = min(n, b + per);
  long long sum = 0;
  for (int i = b; i < e; ++i) {
    sum += lattice_pending(D, chans[i]);
  }
  part[tid] = sum;
  __syncthreads();
  for (int d = 1; d < 1024; d <<= 1) {
    const long long v = tid >= d ? part[tid - d] : 0;
    __syncthreads();
    part[tid] += v;
    __syncthreads();
  }
  long long run = part[tid] - sum;
  for (int i = b; i < e; ++i) {
    offs[i] = run; offs_host[i] = run;
    run += lattice_pending(D, chans[i]);
  }
  if (tid == 1023) { offs[n] = part[1023]; offs_host[n] = part[1023]; }
}
__global__ void k_export_lattice_batch(DecDev D, const int32_t *chans, int n_ch, const long long *offs, LatRec *out, long long cap) {
  if (offs[n_ch] > cap) return;                       // caller's buffer too small: nothing is copied or drained
  const int ch = chans[blockIdx.x];
  const LatInt *lat = D.lat + (size_t)ch * (size_t)D.lat_cap;
  const long long o = offs[blockIdx.x], n = offs[blockIdx.x + 1] - o;
  if (n <= 0) return;
  const long long start = D.chan[ch].lat_head % D.lat_cap;
  for (long long i = (long long)blockIdx.y * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.y * blockDim.x) {
    const LatInt r = lat[start + i < D.lat_cap ? start + i : start + i - D.lat_cap];
    out[o + i] = LatRec{r.frame, D.g.orig[r.arc], r.extra};
  }
}
__global__ void k_reset_lattice_batch(DecDev D, const int32_t *chans, int n, const long long *offs, long long cap) {
  if (offs[n] > cap) return;
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) D.chan[chans[i]].lat_head += offs[i + 1] - offs[i];
}

// The drain of up to DRAIN_FEW channels (what one wavefront scans) in one kernel: every block counts for
// itself, and the last one to finish, when nobody reads the ring positions any more, moves them on.
// (One channel, 30 frames: 14 us in three kernels and the gaps between them, 7 us in one.)
constexpr int DRAIN_FEW = 64;
__global__ void __launch_bounds__(256) k_drain_lattice_few(DecDev D, const int32_t *chans, int n_ch, LatRec *out, long long cap,
                                                           long long *offs_host, uint32_t *finished) {
  __shared__ long long s_first, s_count, s_total;
  __shared__ uint32_t s_before;
  const int tid = threadIdx.x;
  long long mine = 0;                          // (wave 0, one channel per thread)
  if (tid < 64) {
    mine = tid < n_ch ? lattice_pending(D, chans[tid]) : 0;
    long long inc = mine;
    for (int d = 1; d < 64; d <<= 1) {
      const long long v = __shfl_up(inc, d, 64);
      if (tid >= d) inc += v;
    }
    if (tid == (int)blockIdx.x) { s_first = inc - mine; s_count = mine; }
    if (tid == 63) s_total = inc;
    if (blockIdx.x == 0 && blockIdx.y == 0) {
      if (tid < n_ch) offs_host[tid] = inc - mine;
      if (tid == 63) offs_host[n_ch] = inc;
    }
  }
  __syncthreads();
  const bool fits = s_total <= cap;            // (else nothing is copied or drained)
  if (fits && s_count > 0) {
    const int ch = chans[blockIdx.x];
    const LatInt *lat = D.lat + (size_t)ch * (size_t)D.lat_cap;
    const long long o = s_first, n = s_count, start = D.chan[ch].lat_head % D.lat_cap;
    for (long long i = (long long)blockIdx.y * blockDim.x + tid; i < n; i += (long long)gridDim.y * blockDim.x) {
      const LatInt r = lat[start + i < D.lat_cap ? start + i : start + i - D.lat_cap];
      out[o + i] = LatRec{r.frame, D.g.orig[r.arc], r.extra};
    }
  }
  __syncthreads();
  if (tid == 0) s_before = atomicAdd(finished, 1u);
  __syncthreads();
  if (s_before != gridDim.x * gridDim.y - 1u) return;
  if (fits && tid < n_ch) D.chan[chans[tid]].lat_head += mine;
  if (tid == 0) *finished = 0;
}

// Behind a readout's kernels: tells the host, which looks for the number in pinned memory, that they are over.
__global__ void k_signal(uint32_t *done, uint32_t number) { __hip_atomic_store(done, number, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM); }

// Snapshot blocks: the slots of a call's snapshots are emptied before its lanes start.
__global__ void k_reset_blocks(DecDev D, long long id0, int n) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j < n) D.blk[(id0 + j) % D.n_blk] = SnapBlock{0ull, id0 + j};
}
// Where each listed channel's lattice records sit in the block of snapshot `id`:
// out[2i] = start, out[2i+1] = count (0, 0 for a channel without that snapshot);
// out[2n] = records in the block, all lanes together.
__global__ void k_snapshot_ranges(DecDev D, const int32_t *chans, int n, long long id, long long *out) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) {
    const ChanSnap *sp = D.snap + (size_t)chans[i] * SNAP_RING + (size_t)(id % SNAP_RING);
    const bool have = sp->id == id;
    out[2 * i] = have ? sp->blk_start : 0;
    out[2 * i + 1] = have ? sp->blk_count : 0;
  }
  if (i == 0) {
    const SnapBlock b = D.blk[id % D.n_blk];
    out[2 * n] = b.id == id ? (long long)b.used : -1;
  }
}

// ---- final lattice -------------------------------------------------------------------------
// Backward pruning of a channel's buffered lattice arcs with the lattice beam (the paper's
// Section 3.4 leaves this to the end of the utterance).  te(n), the extra cost of token n, is
// the minimum over recorded arcs a: n -> m of te(m) + extra(a); in the last frame it is the
// token's distance to the best (final) cost.  An arc into m is kept iff te(m) + extra(a) <=
// lattice_beam.  fp32, one rounded add per step; minima via integer atomics on the (non-
// negative) float bits, so the result does not depend on thread order.
struct LatticeInfoDev { long long arcs_in, arcs_kept; int32_t frames, reached_final, status, listed; float best_cost, pad2; };

constexpr int FL_NT = 1024;
constexpr int FL_U = 4;                       // records of a frame per thread, in registers
constexpr int FL_TOK = 16384;                 // tokens of a frame whose te fits LDS
constexpr int FL_WIN = 256;                   // frames whose offsets are in LDS at a time
struct FinalShared {
  uint32_t te[2][FL_TOK];
  long long off[FL_WIN + 4], rs[FL_WIN + 4];
  uint32_t changed[3], best_f, best_n, n_list;
  unsigned long long kept;
};

// The pass with te in global memory, frame by frame: for channels with a frame that has more
// tokens than FL_TOK, or more arcs to keep than the list of survivors holds.  Leaves every token's
// te in te[]; returns (to thread 0) the number of arcs kept.
template <class L>
__device__ unsigned long long final_te_global(const DecDev &D, FinalShared &S, L lat, long long n_rec, const long long *foff, int T, long long n_tok,
                                              uint32_t *te, const long long *rec_start, const HTok *hist, bool any_final, float best) {
  const int tid = threadIdx.x, NTH = FL_NT;
  const uint32_t *rec = D.g.rec;
  const long long oT = foff[T];
  const int nT = (int)(foff[T + 1] - oT);
  if (tid == 0) S.kept = 0;
  for (long long i = tid; i < n_tok; i += NTH) te[i] = 0x7F800000u;            // +inf
  __syncthreads();
  for (int i = tid; i < nT; i += NTH) {
    const HTok t = hist[oT + i];
    float v;
    if (any_final) {
      const float fc = __uint_as_float(rec[3 * (size_t)(t.handle & HMASK) + 2]);
      v = fc != INFINITY ? (t.cost + fc) - best : INFINITY;
    } else {
      v = t.cost - best;
    }
    te[oT + i] = __float_as_uint(v);
  }
  __syncthreads();
  for (int f = T; f >= 0; --f) {
    const long long of = foff[f];
    if (f < T) {                                    // emitting arcs recorded with frame f + 1 start in frame f
      const long long of1 = foff[f + 1];
      for (long long i = rec_start[f + 1] + tid; i < rec_start[f + 2]; i += NTH) {
        const LatInt r = lat(i);
        if (r.src & PREV_SAME) continue;
        const float v = __uint_as_float(ld32(&te[of1 + r.dst])) + r.extra;
        atomicMin(&te[of + r.src], __float_as_uint(v));
      }
      __syncthreads();
    }
    const long long e0 = rec_start[f], e1 = rec_start[f + 1];
    for (;;) {                                      // epsilon arcs inside frame f, to the fixed point
      if (tid == 0) S.changed[0] = 0;
      __syncthreads();
      for (long long i = e0 + tid; i < e1; i += NTH) {
        const LatInt r = lat(i);
        if (!(r.src & PREV_SAME)) continue;
        const uint32_t v = __float_as_uint(__uint_as_float(ld32(&te[of + r.dst])) + r.extra);
        if (v < atomicMin(&te[of + (r.src & ~PREV_SAME)], v)) S.changed[0] = 1;
      }
      __syncthreads();
      if (!S.changed[0]) break;
      __syncthreads();
    }
  }
  unsigned long long kept = 0;
  for (long long i = tid; i < n_rec; i += NTH) {
    const LatInt r = lat(i);
    const float v = __uint_as_float(ld32(&te[foff[r.frame] + r.dst])) + r.extra;
    kept += v <= D.lattice_beam ? 1 : 0;
  }
  if (kept) atomicAdd(&S.kept, kept);
  __syncthreads();
  return S.kept;
}

// Pass 1, one workgroup per listed channel.  The channel's scratch: te, one word per token, and
// rec_start, one offset per frame; te_stride / rs_stride: distance between the scratch areas of
// consecutive channel ids (0: a single area, for a call on one channel).
//
// The frames are a serial chain, so what counts is the time per frame.  te of two frames lives in
// LDS; a frame's records are in registers, requested two frames ahead; candidates beyond the
// lattice beam are dropped at once (extra costs are not negative: nothing kept can come of them),
// which leaves a few dozen live tokens per frame; two barriers per frame plus one per further
// round over the epsilon arcs.  The surviving arcs are listed as they are found (in the te scratch,
// which this form does not need), so no second pass over all records is made.
// With te in global memory, one pass over all records to find the frames, one to count and one to
// emit, the whole call took 2.31 ms for a 300-frame stream on the 1000-state graph, 13.6 ms for 400
// frames of 6600 arcs and 11.8 ms for 100 utterances of 500 - 1500 frames; now 0.51, 1.71, 2.12 ms.
__global__ void __launch_bounds__(FL_NT) k_final_lattice_te(DecDev D, const int32_t *chans, int use_final, uint32_t *te_base,
                                                            long long te_stride, long long *rs_base, long long rs_stride,
                                                            LatticeInfoDev *info) {
  __shared__ FinalShared S;
  const int tid = threadIdx.x, lane = tid & 63;
  const int ch = chans[blockIdx.x];
  uint32_t *list = te_base + (size_t)ch * (size_t)te_stride;
  long long *rec_start = rs_base + (size_t)ch * (size_t)rs_stride;
  const ChanState *cs = D.chan + ch;
  const long long *foff = D.frame_off + (size_t)ch * (size_t)(D.max_frames + 2);
  const HTok *hist = D.hist + (size_t)ch * (size_t)D.hist_cap;
  const LatInt *lat_ring = D.lat + (size_t)ch * (size_t)D.lat_cap;
  const long long lat_first = cs->lat_head % D.lat_cap, lat_cap = D.lat_cap;
  // record i of the buffered ones (they start at ring position lat_first)
  auto lat = [&](long long i) -> const LatInt & { return lat_ring[lat_first + i < lat_cap ? lat_first + i : lat_first + i - lat_cap]; };
  const uint32_t *rec = D.g.rec;
  const int st = cs->status;
  const bool readable = st == 0;
  const int T = cs->num_frames - 1;
  const long long n_rec = cs->lat_total - cs->lat_head;
  const long long n_tok = cs->hist_used;
  const long long oT = T >= 0 ? foff[T] : 0;
  const int nT = T >= 0 ? (int)(foff[T + 1] - oT) : 0;
  if (!readable || nT == 0) {
    if (tid == 0) { LatticeInfoDev li{n_rec, 0, T + 1, 0, readable ? E_DEAD_CHANNEL : st, 0, 0.f, 0.f}; info[blockIdx.x] = li; }
    return;
  }
  if (tid == 0) { S.best_f = KEY_NONE; S.best_n = KEY_NONE; S.n_list = 0; S.changed[0] = 0; S.changed[1] = 0; S.changed[2] = 0; }
  // where each frame's run of records starts (they are appended frame by frame), by bisection
  for (int f = tid; f <= T + 2; f += FL_NT) {
    long long lo = 0, hi = n_rec;
    while (lo < hi) {
      const long long mid = (lo + hi) >> 1;
      if (lat(mid).frame < f) lo = mid + 1; else hi = mid;
    }
    rec_start[f] = lo;
  }
  __syncthreads();
  // best cost over the last frame
  {
    uint32_t bn = KEY_NONE, bf = KEY_NONE;
    for (int i = tid; i < nT; i += FL_NT) {
      const HTok t = hist[oT + i];
      bn = min(bn, okey(t.cost));
      if (use_final) {
        const float fc = __uint_as_float(rec[3 * (size_t)(t.handle & HMASK) + 2]);
        if (fc != INFINITY) bf = min(bf, okey(t.cost + fc));
      }
    }
    bn = wave_min_u32(bn); bf = wave_min_u32(bf);
    if (lane == 0) { atomicMin(&S.best_n, bn); atomicMin(&S.best_f, bf); }
  }
  __syncthreads();
  const bool any_final = use_final && S.best_f != KEY_NONE;
  const float best = key2f(any_final ? S.best_f : S.best_n);
  const float beam = D.lattice_beam;
  bool in_lds = cs->max_post <= FL_TOK && n_rec < 0xFFFFFFFFll;
  if (in_lds) {
    for (int i = tid; i < nT; i += FL_NT) {
      const HTok t = hist[oT + i];
      float v;
      if (any_final) {
        const float fc = __uint_as_float(rec[3 * (size_t)(t.handle & HMASK) + 2]);
        v = fc != INFINITY ? (t.cost + fc) - best : INFINITY;
      } else {
        v = t.cost - best;
      }
      S.te[T & 1][i] = __float_as_uint(v);
    }
    int w0 = 0;                                     // first frame of the window of offsets
    auto load_window = [&](int top) {               // (frames top + 1 and below)
      __syncthreads();
      w0 = max(0, top + 2 - FL_WIN);
      for (int i = tid; i < FL_WIN + 4; i += FL_NT) {
        const int f = w0 + i;
        S.off[i] = f <= T + 1 ? foff[f] : 0;
        S.rs[i] = f <= T + 2 ? rec_start[f] : n_rec;
      }
      __syncthreads();
    };
    load_window(T);
    struct Rec { float extra; uint32_t dst, src; };
    struct Recs { Rec r[FL_U]; };
    auto request = [&](int f, Recs &q) {            // the records of frame f that this thread holds in registers
      const long long a = f >= 0 ? S.rs[f - w0] : 0, b = f >= 0 ? S.rs[f + 1 - w0] : 0;
#pragma unroll
      for (int u = 0; u < FL_U; ++u) {
        const long long i = a + u * FL_NT + tid;
        if (i < b) { const LatInt &l = lat(i); q.r[u].extra = l.extra; q.r[u].dst = l.dst; q.r[u].src = l.src; }
      }
    };
    uint32_t round = 0;                             // rounds over epsilon arcs so far, all frames
    auto step = [&](int f, const Recs &q) {
      const long long a = S.rs[f - w0], b = S.rs[f + 1 - w0];
      const int n_below = f > 0 ? (int)(S.off[f - w0] - S.off[f - 1 - w0]) : 0;
      uint32_t *cur = S.te[f & 1], *below = S.te[(f & 1) ^ 1];
      for (int i = tid; i < n_below; i += FL_NT) below[i] = 0x7F800000u;
      auto each = [&](auto fn) {
#pragma unroll
        for (int u = 0; u < FL_U; ++u) {
          const long long i = a + u * FL_NT + tid;
          if (a + u * FL_NT < b) fn(i < b, i, q.r[u]);
        }
#pragma unroll 1
        for (long long i0 = a + FL_U * FL_NT; i0 < b; i0 += FL_NT) {
          const long long i = i0 + tid;
          Rec r{0.f, 0, 0};
          if (i < b) { const LatInt &l = lat(i); r = Rec{l.extra, l.dst, l.src}; }
          fn(i < b, i, r);
        }
      };
      for (;;) {                                    // epsilon arcs inside the frame, to the fixed point
        if (tid == 0) S.changed[(round + 1) % 3] = 0;
        each([&](bool mine, long long, const Rec &r) {
          if (!mine || !(r.src & PREV_SAME)) return;
          const float v = __uint_as_float(cur[r.dst]) + r.extra;
          if (v <= beam && __float_as_uint(v) < atomicMin(&cur[r.src & ~PREV_SAME], __float_as_uint(v))) S.changed[round % 3] = 1;
        });
        lds_barrier();
        if (!uni(S.changed[round++ % 3])) break;
      }
      each([&](bool mine, long long i, const Rec &r) {
        const float v = mine ? __uint_as_float(cur[r.dst]) + r.extra : INFINITY;
        const bool keep = v <= beam;
        if (keep && !(r.src & PREV_SAME)) atomicMin(&below[r.src], __float_as_uint(v));
        const unsigned long long m = __ballot(keep);
        if (m) {
          uint32_t p = 0;
          if (lane == 0) p = atomicAdd(&S.n_list, (uint32_t)__popcll(m));
          p = uni(p) + (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
          if (keep && (long long)p < n_tok) list[p] = (uint32_t)i;
        }
      });
      lds_barrier();
    };
    Recs q0, q1, q2;
    request(T, q0); request(T - 1, q1);
    for (int f = T; f >= 0;) {
      if (f < w0 + 6 && w0 > 0) load_window(f);     // (three steps, each looking three frames down)
      request(f - 2, q2); step(f, q0); --f;
      if (f < 0) break;
      request(f - 2, q0); step(f, q1); --f;
      if (f < 0) break;
      request(f - 2, q1); step(f, q2); --f;
    }
    if ((long long)S.n_list > n_tok) in_lds = false;        // (more survivors than the list holds)
    __syncthreads();
  }
  unsigned long long kept = S.n_list;
  if (!in_lds) kept = final_te_global(D, S, lat, n_rec, foff, T, n_tok, list, rec_start, hist, any_final, best);
  if (tid == 0) {
    LatticeInfoDev li{n_rec, (long long)kept, T + 1, any_final ? 1 : 0, 0, in_lds ? 1 : 0, best, 0.f};
    info[blockIdx.x] = li;
  }
}

// offs[0..n]: exclusive prefix sums of the kept-arc counts of pass 1 (one block); they and the
// channels' results also go straight to pinned host memory.
__global__ void __launch_bounds__(1024) k_final_lattice_offsets(const LatticeInfoDev *info, int n, long long *offs, long long *offs_host,
                                                                LatticeInfoDev *info_host) {
  __shared__ long long part[1024];
  const int tid = threadIdx.x;
  const int per = (n + 1023) / 1024;
  const int b = tid * per, e = min(n, b + per);
  long long sum = 0;
  for (int i = b; i < e; ++i) sum += info[i].status == 0 ? info[i].arcs_kept : 0;
  part[tid] = sum;
  __syncthreads();
  for (int d = 1; d < 1024; d <<= 1) {
    const long long v = tid >= d ? part[tid - d] : 0;
    __syncthreads();
    part[tid] += v;
    __syncthreads();
  }
  long long run = part[tid] - sum;
  for (int i = b; i < e; ++i) {
    const LatticeInfoDev li = info[i];
    offs[i] = run; offs_host[i] = run; info_host[i] = li;
    run += li.status == 0 ? li.arcs_kept : 0;
  }
  if (tid == 1023) { offs[n] = part[1023]; offs_host[n] = part[1023]; }
}

// Pass 2: the surviving arcs of listed channel blockIdx.x, in the caller's form, at out[offs[blockIdx.x] ..).
// Nothing is written if the caller's buffer cannot take all channels' arcs.
__global__ void __launch_bounds__(1024) k_final_lattice_emit(DecDev D, const int32_t *chans, int n_ch, const uint32_t *te_base,
                                                             long long te_stride, const long long *offs, LatRec *out,
                                                             long long cap, const LatticeInfoDev *info) {
  if (offs[n_ch] > cap || info[blockIdx.x].status != 0) return;
  const int tid = threadIdx.x, NTH = 1024;
  const int ch = chans[blockIdx.x];
  const uint32_t *te = te_base + (size_t)ch * (size_t)te_stride;
  const ChanState *cs = D.chan + ch;
  const long long *foff = D.frame_off + (size_t)ch * (size_t)(D.max_frames + 2);
  const LatInt *lat_ring = D.lat + (size_t)ch * (size_t)D.lat_cap;
  const long long lat_first = cs->lat_head % D.lat_cap, lat_cap = D.lat_cap;
  const long long n_rec = cs->lat_total - cs->lat_head;
  LatRec *dst = out + offs[blockIdx.x];
  auto lat = [&](long long i) -> const LatInt & { return lat_ring[lat_first + i < lat_cap ? lat_first + i : lat_first + i - lat_cap]; };
  if (info[blockIdx.x].listed) {                    // te[] holds the numbers of the surviving records
    const long long n = info[blockIdx.x].arcs_kept;
    for (long long i = tid; i < n; i += NTH) {
      const LatInt &r = lat((long long)te[i]);
      dst[i] = LatRec{r.frame, D.g.orig[r.arc], r.extra};
    }
    return;
  }
  __shared__ unsigned long long s_pos;
  if (tid == 0) s_pos = 0;
  __syncthreads();
  for (long long i = tid; i < n_rec; i += NTH) {
    const LatInt r = lat(i);
    const float v = __uint_as_float(te[foff[r.frame] + r.dst]) + r.extra;
    if (v <= D.lattice_beam) {
      const unsigned long long p = atomicAdd(&s_pos, 1ull);
      dst[p] = LatRec{r.frame, D.g.orig[r.arc], r.extra};
    }
  }
}

}  // namespace wfst
