// What the forms of a lane's frame share: cost keys, the state table, wavefront and workgroup
// primitives, and the LDS block of a lane.
#pragma once
#include "wfst_device.h"

namespace wfst {

constexpr int NBINS = 1024;
// ---- wavefront primitives (all 64 lanes must be active) ------------------------------------
template <int CTRL> __device__ __forceinline__ int dpp_mov(int old, int v) {
  return __builtin_amdgcn_update_dpp(old, v, CTRL, 0xF, 0xF, false);
}
// inclusive prefix sum over the wavefront
__device__ __forceinline__ int wave_incl_scan(int v) {
  v += dpp_mov<0x111>(0, v);                 // row_shr:1, lanes without a source add 0
  v += dpp_mov<0x112>(0, v);
  v += dpp_mov<0x114>(0, v);
  v += dpp_mov<0x118>(0, v);                 // inclusive within each row of 16
  const int t0 = __builtin_amdgcn_readlane(v, 15), t1 = __builtin_amdgcn_readlane(v, 31), t2 = __builtin_amdgcn_readlane(v, 47);
  const int row = (threadIdx.x & 63) >> 4;
  return v + (row >= 1 ? t0 : 0) + (row >= 2 ? t1 : 0) + (row >= 3 ? t2 : 0);
}
__device__ __forceinline__ uint32_t wave_min_u32(uint32_t v) {
  v = min(v, (uint32_t)dpp_mov<0x111>((int)v, (int)v));
  v = min(v, (uint32_t)dpp_mov<0x112>((int)v, (int)v));
  v = min(v, (uint32_t)dpp_mov<0x114>((int)v, (int)v));
  v = min(v, (uint32_t)dpp_mov<0x118>((int)v, (int)v));      // lane 15 of each row: the row's minimum
  const uint32_t a = (uint32_t)__builtin_amdgcn_readlane((int)v, 15), b = (uint32_t)__builtin_amdgcn_readlane((int)v, 31);
  const uint32_t c = (uint32_t)__builtin_amdgcn_readlane((int)v, 47), d = (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
  return min(min(a, b), min(c, d));
}
// One counter update per wavefront: the lanes that call this together (same call site, any
// subset of the wave) get consecutive indices from a single atomic add.
__device__ __forceinline__ uint32_t wave_alloc(uint32_t *counter) {
  const unsigned long long m = __ballot(1);
  const int lane = threadIdx.x & 63;
  const int leader = __ffsll((long long)m) - 1;
  uint32_t base = 0;
  if (lane == leader) base = atomicAdd(counter, (uint32_t)__popcll(m));
  base = (uint32_t)__builtin_amdgcn_readlane((int)base, leader);
  return base + (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
}
// Fetch ahead: start the load of the line that holds *p without waiting for it and without
// tying up a register - the value is delivered to a scratch word in LDS (`sink`: the LDS
// address of 64 floats nobody reads) by the LDS-direct form of the load.  A later ordinary
// load of the same line finds it in the cache or on its way.  The compiler does not count this
// load in its vmcnt bookkeeping; since vector memory operations complete in order, the waits
// it inserts for its own loads stay correct (an older operation in the queue can only make
// them wait for slightly more than they need).
__device__ __forceinline__ void fetch_ahead(const void *p, uint32_t sink) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %0, off" ::"v"(p), "s"(sink) : "m0", "memory");
}
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// ---- LDS structures of a light frame ----------------------------------------------------------
// A 512-thread lane shares its compute unit's 160 KB of LDS with another lane; a 1024-thread
// lane has the unit to itself and takes structures twice as large.
template <int NT> struct LightCfg {
  static constexpr int SLOTS = NT >= 1024 ? 4096 : 2048;   // state table
  static constexpr int HBITS = NT >= 1024 ? 12 : 11;
  static constexpr int CLAIM_LIMIT = SLOTS * 3 / 4;        // states reached in a frame = tokens of the next one
  static constexpr int TILE = NT * 4;                      // emitting arcs expanded together, four per thread
  static constexpr int ARCS = TILE * 2;                    // emitting arcs of a frame
  static constexpr int MARK_WORDS = ARCS / 32;
  static constexpr int ECAP = NT >= 1024 ? 2560 : 1280;    // epsilon arcs listed in a frame
  static constexpr uint32_t MAX_PROBES = 256;              // of the table (a frame that fills it is given up)
};
// Slot::aux of the light table: degree info of the state << 16 | index of its token in the new
// frame (POS_NONE: cut by max-active)
constexpr uint32_t POS_NONE = 0xFFFFu;
constexpr uint32_t TOK_DEAD = 0x80000000u;    // in LaneShared::tok: the state has no emitting arc (it takes one arc position all the same)
constexpr uint32_t EA_AGAIN = 0x8000u, EA_SLOT = 0x7FFFu;  // epsilon entry: listed before, its source has improved since
// What a stage allots, one 64-bit counter: [63] give the frame up, [62:32] arc positions of the
// next frame, [31:16] epsilon arcs listed, [15:0] states claimed
constexpr unsigned long long CNT_RESTART = 1ull << 63;
constexpr int CNT_ARC_SHIFT = 32, CNT_EPS_SHIFT = 16;
constexpr uint32_t CNT_ARCS = 0x7FFFFFFFu;
constexpr uint32_t F_NAN = 1, F_TOKOVF = 2, F_LATOVF = 4;
constexpr uint32_t KEY_NONE = 0xFFFFFFFFu;
constexpr uint32_t KEY_PINF = 0xFF800000u;    // okey(+inf)

// Counters of one frame.  Two sets are used alternately, so that a frame can start while the
// previous frame's values are still being read; the set not in use is reset in between.
struct __align__(16) FrameCtr {
  // what the insertion and the closure rounds allot.  A round's counter is final at the round's
  // barrier (the next round uses another one), so every thread reads the same value there - also
  // the request to give the frame up.
  unsigned long long cnt[3];
  unsigned long long sel;      // after a selection: arc positions << 32 | tokens kept
  uint32_t flags, latn, dead, again;   // (read together at the end of the frame)
  uint32_t best, kmin, kmax, pad;
};
__device__ __forceinline__ void reset_ctr(FrameCtr &c) {
  c.cnt[0] = 0; c.cnt[1] = 0; c.cnt[2] = 0; c.sel = 0;
  c.best = KEY_NONE; c.flags = 0; c.latn = 0; c.dead = 0; c.again = 0;
  c.kmin = 0xFFFFFFFFu; c.kmax = 0;
}

// State of a lane that every thread of its workgroup holds in registers (all values uniform; as
// little as possible, since scalar registers are what the light frame runs out of).  What is only
// counted is in LDS (LaneShared::arcs_expanded, max_pre, max_post, iters_max), kept by one thread.
struct LaneCtx {
  int status, nf;
  int n_in;                  // tokens of the last frame: [hist_used - n_in, hist_used) of the history
  long long hist_used;
  long long lat_total;       // lattice records produced since init,
  long long lat_pend;        //   of which not handed out yet,
  long long lat_pos;         //   and the ring position of the next one
  uint32_t pending_clear;    // states claimed by the last light frame, whose table slots are still to be cleared
  int par;                   // counter set (and set of first-arc marks) the next light frame uses
  bool lds_foreign;          // a heavy frame has used the light frame's place in LDS
  bool tok_valid;            // the LDS token list holds the frame the next one starts from:
  uint32_t n_arcs, n_dead;   // arc positions its tokens take, and how many of them belong to tokens without an emitting arc
#ifdef WFST_PHASE_TIMING
  unsigned long long tlast;
#endif
};
// A value every lane of the wavefront holds alike, moved to a scalar register (values that
// come from LDS or from vector loads sit in vector registers otherwise, and so would
// everything computed from them: the lane's whole state and its arithmetic).
__device__ __forceinline__ uint32_t uni(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ unsigned long long uni(unsigned long long v) {
  return ((unsigned long long)uni((uint32_t)(v >> 32)) << 32) | uni((uint32_t)v);
}
__device__ __forceinline__ long long uni(long long v) { return (long long)uni((unsigned long long)v); }
// (a row of scores: named as global memory, or what is loaded through it would be taken for generic)
__device__ __forceinline__ const float *uni(const float *p) {
  return (const float *)(__attribute__((address_space(1))) const float *)uni((unsigned long long)p);
}
__device__ __forceinline__ float uni(float v) { return __uint_as_float(uni(__float_as_uint(v))); }


__device__ __forceinline__ uint32_t okey(float x) {
  uint32_t b = __float_as_uint(x);
  return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}
__device__ __forceinline__ float key2f(uint32_t k) {
  return __uint_as_float((k & 0x80000000u) ? (k & 0x7FFFFFFFu) : ~k);
}
__device__ __forceinline__ unsigned long long pack(uint32_t key, uint32_t arc) {
  return ((unsigned long long)key << 32) | arc;
}
// Loads that bypass the per-CU vector cache: table words are updated by atomics, which
// execute in L2, so cached copies could be stale.
__device__ __forceinline__ uint32_t ld32(const uint32_t *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long ld64(const unsigned long long *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint32_t slot_hash(uint32_t handle, int hbits) {
  return (handle * 2654435761u) >> (32 - hbits);
}
// Where a table in LDS is looked into next for a state whose slot another one has: an odd step of the
// state's own, which comes past every slot of the table.  The tables fill up to three quarters, and a
// wave is as slow as its unluckiest candidate: going on to the next slot, the longest of a wave's 256
// searches took 16.5 probes with 3000 states in 4096 slots, and the longest of the frame 58; with this
// 7.6 and 18 (500 states in 2048: 3.8 and 3.3 for a wave).  Whole calls, slot by slot and this, us: 64 streams of a
// wide beam with an approximate limit of 2000 11196 -> 9202, 150 of beam 18 9219 -> 8662, 100 of beam 15
// 20706 -> 20290, 500 of beam 13 10705 -> 10559; one stream of few tokens 3108 and 3136 -> 3152 and 3185 (two
// runs of each).  One stream of very many tokens, a team of eight, is not decided: its runs come in two kinds,
// 30.5 - 30.8 and 32.4 - 32.6 ms, and of four slot by slot one was of the second, of two with this both.
// (The table in memory, which is at most half full, is searched slot by slot.)
__device__ __forceinline__ uint32_t slot_step(uint32_t handle) { return ((handle * 2654435761u) >> 6) | 1u; }

// Table words are read through these: in global memory with loads that bypass the per-CU
// vector cache (see ld32), in LDS with plain loads.
template <bool LDS> __device__ __forceinline__ uint32_t tl32(const uint32_t *p) { return LDS ? *p : ld32(p); }
template <bool LDS> __device__ __forceinline__ unsigned long long tl64(const unsigned long long *p) { return LDS ? *p : ld64(p); }

// Offer candidate K for state `handle`.  Returns the slot, or -1 if the table is full.
template <bool LDS>
__device__ __forceinline__ int ht_insert(Slot *slots, uint32_t mask, int hbits, uint32_t handle,
                                         unsigned long long K, bool &claimed, bool &improved) {
  uint32_t h = slot_hash(handle, hbits);
  const uint32_t step = LDS ? slot_step(handle) : 1u;      // (as ht_find looks for it)
  claimed = false; improved = false;
  for (uint32_t probe = 0; probe <= mask; ++probe) {
    // one compare-and-swap tells all three cases apart: free (now ours), ours already, another state's
    uint32_t k = atomicCAS(&slots[h].handle, EMPTY, handle);
    if (k == EMPTY) { claimed = true; k = handle; }
    if (k == handle) {
      unsigned long long old = atomicMin(&slots[h].val, K);
      improved = K < old;
      return (int)h;
    }
    h = (h + step) & mask;
  }
  return -1;
}
// A whole slot at once: in LDS one 16-byte read instead of dependent 8- and 4-byte ones (a
// reader beside concurrent atomic minima gets some value the slot held, which is all the
// callers need); in global memory three independent coherent loads.
template <bool LDS>
__device__ __forceinline__ Slot ld_slot(const Slot *p) {
  Slot r;
  if (LDS) {
    *reinterpret_cast<uint4 *>(&r) = *reinterpret_cast<const uint4 *>(p);
  } else {
    r.val = ld64(&p->val); r.handle = ld32(&p->handle); r.aux = ld32(&p->aux);
  }
  return r;
}
template <bool LDS>
__device__ __forceinline__ int ht_find(const Slot *slots, uint32_t mask, int hbits, uint32_t handle) {
  uint32_t h = slot_hash(handle, hbits);
  const uint32_t step = LDS ? slot_step(handle) : 1u;
  for (uint32_t probe = 0; probe <= mask; ++probe) {
    uint32_t k = tl32<LDS>(&slots[h].handle);
    if (k == handle) return (int)h;
    if (k == EMPTY) return -1;
    h = (h + step) & mask;
  }
  return -1;
}

constexpr int EXP_U = 4;                   // general frame: arcs per thread and round of the emitting expansion
constexpr int EPS_U = 2;                   // epsilon arcs of a token fetched together
constexpr int LAT_U = 4;                   // candidate records per thread and round of the lattice stage
constexpr uint32_t AUX_EPS = 0x80000000u;  // Aux::slot flag: the record is an epsilon arc
// Slot::aux of the general frame while a frame is being built (afterwards: index of the kept token, or ~0):
constexpr uint32_t A_FRESH = 0x80000000u;  // epsilon out-degree not counted yet
constexpr uint32_t A_KEPT_MAX = 0x20000000u;  // aux < A_KEPT_MAX: index of the kept token

// Counters of a general frame (the lane's first workgroup works through it alone).
struct GenCtr {
  // queue entries (low word) and states claimed (high word) of the frame: one 64-bit counter,
  // so that a claim takes one atomic for both
  unsigned long long claim_ctr;
  unsigned long long emit_arcs, eps_arcs;
  uint32_t auxn, best, flags, nvalid, nout, latn, kmin, kmax;
};
// ---- heavy frames (see wfst_frame_heavy.h) -----------------------------------------------------
constexpr int TEAM_MAX = 16;                  // workgroups of a lane
constexpr int HEAVY_LIST = 512;               // (cost, state) pairs that the selection ranks one against the other
template <int NT> struct HeavyCfg {
  static constexpr int SLOTS = NT >= 1024 ? 8192 : 4096;   // state table of a workgroup: all the LDS there is
  static constexpr int HBITS = NT >= 1024 ? 13 : 12;
  static constexpr int CLAIM_LIMIT = SLOTS * 3 / 4;
  static constexpr uint32_t MAX_PROBES = 256;
};
constexpr uint32_t EL_AGAIN = 0x80000000u;    // in a list of epsilon arcs: listed before, its source has improved since
constexpr uint32_t EV_FAIL = 0x80000000u, EV_NAN = 0x40000000u, EV_LATOVF = 0x20000000u, EV_COUNT = 0x0FFFFFFFu;
// What the workgroups of a heavy frame share: in LDS when there is one, in global memory when
// there are several (then read with loads that bypass the vector cache).
template <int M> struct HeavyCtr {
  uint32_t ev[3];              // events of a barrier, and how many candidates were sent before it
  uint32_t best, nout, latn, kmax, listed;
  unsigned long long emit[M];  // emitting arcs expanded
  uint32_t eps[M];             // epsilon out-degrees of the tokens within the beam
  uint32_t claims[2][M];       // states entered so far (two sets, used at alternate barriers, as the next)
  uint32_t cnt[2][M][M];       // [owner][sender]: candidates in the bucket
};
template <int M> __device__ __forceinline__ void reset_heavy(HeavyCtr<M> &c) {
  c.ev[0] = 0; c.ev[1] = 0; c.ev[2] = 0;
  c.best = KEY_NONE; c.nout = 0; c.latn = 0; c.kmax = 0; c.listed = 0;
}
struct HeavyState {            // of the lane, as a heavy frame starts from it
  const float *ll;
  long long in_off, hist_used, lat_pos, lat_room;
  int nf, n_in;
};
struct HeavyLocal {            // one workgroup's own counters, in LDS
  unsigned long long ctr;      // epsilon arcs listed << 32 | states claimed
  uint32_t best, again, fail, lat_full, kept, sent, pos0, pad;
  uint32_t to[TEAM_MAX];       // candidates put into each owner's bucket
  uint32_t from[TEAM_MAX], upto[TEAM_MAX];   // of each sender: candidates taken before, and now
  uint32_t emitted[TEAM_MAX];  // of each sender: emitting candidates
};
// A lane with several workgroups, in global memory.
constexpr unsigned long long TEAM_CLOSED = 1ull << 31;
enum { TEAM_FRAME = 1, TEAM_EXIT = 2 };
struct TeamLane {
  unsigned long long join;     // launch << 32 | TEAM_CLOSED | workgroups that have joined
  uint32_t xcc_mask;           // the XCDs they run on
  uint32_t cmd_seq, cmd;       // commands given so far, and the last one
  uint32_t arrived, broken;    // barriers
  uint32_t G, same_xcd;
  HeavyState hs;
  HeavyCtr<TEAM_MAX> ctr[2];   // used by alternate frames
  uint32_t hist[3][NBINS];     // the selection's passes rotate through three histograms: pass p counts into
                               // p % 3 and zeroes (p + 2) % 3, which nobody reads any more
};

struct TeamCtx {               // a workgroup's place in its lane's team, in its LDS
  TeamLane *tl;
  int g, G;                    // its number, and how many there are
  uint32_t epoch;              // arrivals expected at the next barrier (thread 0 keeps count)
  uint32_t spin_limit;
  uint32_t seq;                // frames the team has worked through
  uint32_t pass;               // histogram passes so far (same in all workgroups)
  uint32_t same_xcd;
  uint32_t commands;           // of the lane's first workgroup, seen so far
};

// LDS of a lane's workgroup.
template <int NT>
struct LaneShared {
  int wave_tmp[NT / 64];
  int wtot[NT / 64];
  float sink[64];              // where fetch_ahead delivers; never read
  union {                      // the expansion's tile arrays and the selection's histogram never coexist
    struct { int scan[NT]; float cost[NT]; uint32_t base[NT]; };
    uint32_t hist[NBINS];
  };
  // -- general frame: its counters, and the lane's state while such a frame runs (between light
  //    frames the state lives in registers, see LaneCtx)
  GenCtr gen;
  uint32_t sel_bin, sel_below, sel_cnt;
  int status, nf, max_pre, max_post, iters_max, n_in;
  long long in_off, hist_used, lat_room, lat_total, arcs_expanded;
  long long lat_pos;           // ring position of record number lat_total
  long long blk_pos;           // seal scratch
#ifdef WFST_PHASE_TIMING
  unsigned long long ph[16], gph[16], gtlast, dbg_tok, dbg_iters, dbg_arcs;
#endif
  FrameCtr fc[2];              // light frames
  uint32_t list_dead;
  HeavyCtr<1> hc;              // heavy frames
  HeavyLocal hl;
  HeavyState hs;
  TeamCtx team;
  uint32_t team_ok, team_cmd;
  unsigned long long sel_theta;
  union {
    struct {                   // -- light frame
      uint2 tok[LightCfg<NT>::CLAIM_LIMIT];        // kept tokens of the last frame = queue of the next: state handle | TOK_DEAD, cost
      uint16_t tok_a[LightCfg<NT>::CLAIM_LIMIT];   //   position of the token's first arc among the frame's arcs
      uint2 mark[2][LightCfg<NT>::MARK_WORDS];     // arc positions at which a token's arcs begin (bits), and their number in the words before
      uint16_t lq[LightCfg<NT>::CLAIM_LIMIT];      // claimed slots, in the order of their tokens
      uint32_t ea_r[LightCfg<NT>::ECAP];           // epsilon arcs to relax: arc,
      float ea_w[LightCfg<NT>::ECAP];              //   weight (once fetched),
      uint16_t ea_s[LightCfg<NT>::ECAP];           //   slot of the source | EA_AGAIN,
      uint16_t ea_d[LightCfg<NT>::ECAP];           //   slot of the destination, 0xFFFF if the candidate was beyond the cutoff
      Slot table[LightCfg<NT>::SLOTS];             // state table
    };
    struct {                   // -- heavy frame
      Slot table[HeavyCfg<NT>::SLOTS];
      uint16_t lq[HeavyCfg<NT>::CLAIM_LIMIT];      // claimed slots
    } hv;
  };
};

// The workgroup's LDS block.  (Functions that are not inlined name it themselves: a reference
// handed to them would be a generic pointer.)
template <int NT, bool TEAM> __device__ __forceinline__ LaneShared<NT> &lane_lds() {
  static __shared__ LaneShared<NT> S;
  return S;
}

#ifdef WFST_PHASE_TIMING
// (instrumented builds) thread 0 adds the time since its previous mark to phase k
#define PHASE_MARK(k) do { if (threadIdx.x == 0) { unsigned long long t_ = wall_clock64(); atomicAdd(&S.ph[k], t_ - ctx.tlast); ctx.tlast = t_; } } while (0)
#else
#define PHASE_MARK(k) do { } while (0)
#endif
#ifdef WFST_PHASE_TIMING
#define GEN_MARK(k) do { if (threadIdx.x == 0) { unsigned long long t_ = wall_clock64(); S.gph[k] += t_ - S.gtlast; S.gtlast = t_; } } while (0)
#else
#define GEN_MARK(k) do { } while (0)
#endif

// Workgroup barrier for stages that communicate through LDS only: it orders LDS accesses but
// does not wait for global loads or stores in flight, so the score-row touch and the stores of
// notes / tokens / lattice records keep travelling across it.  With LOCAL false it is an
// ordinary __syncthreads() (the global-table path communicates through global memory).
template <bool LOCAL>
__device__ __forceinline__ void wg_sync() {
  if (LOCAL) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
  } else {
    __syncthreads();
  }
}

template <int NT, bool LOCAL = false>
__device__ __forceinline__ int block_excl_scan(int v, int *s_wave, int &total) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  int inc = v;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    int t = __shfl_up(inc, d, 64);
    if (lane >= d) inc += t;
  }
  if (lane == 63) s_wave[wid] = inc;
  wg_sync<LOCAL>();
  int base = 0, tot = 0;
#pragma unroll
  for (int i = 0; i < NT / 64; ++i) {
    int t = s_wave[i];
    if (i < wid) base += t;
    tot += t;
  }
  wg_sync<LOCAL>();
  total = tot;
  return base + inc - v;
}

// The need-th smallest (1-based) of the values val(i, v) accepts, all known to lie in
// [lo, hi]: theta, with the number of accepted values below it and equal to it.  Exact:
// only integer histograms, refined until a bin is one value wide.
template <int NT, class F>
__device__ void block_select(LaneShared<NT> &S, int n, uint32_t need, uint32_t lo, uint32_t hi, F val,
                             uint32_t &theta, uint32_t &n_less, uint32_t &n_eq) {
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));            // (what depends on it is computed here, not held in registers all through the kernel)
  constexpr int PER = NBINS / NT;
  uint32_t less = 0;
  for (;;) {
    int shift = 0;                           // bins of 2^shift values: the last value, hi, must fall into bin NBINS - 1 at most
    while ((((unsigned long long)hi - lo) >> shift) >= (unsigned long long)NBINS) ++shift;
    for (int b = tid; b < NBINS; b += NT) S.hist[b] = 0;
    __syncthreads();
    for (int i = tid; i < n; i += NT) {
      uint32_t v;
      if (val(i, v) && v >= lo && v <= hi) atomicAdd(&S.hist[(v - lo) >> shift], 1u);
    }
    __syncthreads();
    uint32_t loc[PER], sum = 0;
#pragma unroll
    for (int q = 0; q < PER; ++q) { loc[q] = S.hist[tid * PER + q]; sum += loc[q]; }
    int total;
    uint32_t run = (uint32_t)block_excl_scan<NT>((int)sum, S.wave_tmp, total);
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      if (run < need && run + loc[q] >= need) { S.sel_bin = tid * PER + q; S.sel_below = run; S.sel_cnt = loc[q]; }
      run += loc[q];
    }
    __syncthreads();
    const uint32_t b = S.sel_bin, below = S.sel_below, cnt = S.sel_cnt;
    __syncthreads();
    less += below;
    need -= below;
    lo = lo + (b << shift);
    unsigned long long nhi = (unsigned long long)lo + ((1ull << shift) - 1);
    if (nhi < hi) hi = (uint32_t)nhi;
    if (shift == 0) { theta = lo; n_less = less; n_eq = cnt; return; }
  }
}

// The approximate form of the selection (the paper's histogram-based max-active, Section 4.1):
// ONE histogram of NBINS equal-width bins over [lo, hi]; the cut is the upper edge of the bin in
// which the running count reaches `need`, so up to that bin's population more than `need`
// values lie at or below it.  Integer counting only: the same cut whatever the thread order.
template <int NT, class F>
__device__ uint32_t block_histogram_cut(LaneShared<NT> &S, int n, uint32_t need, uint32_t lo, uint32_t hi, F val) {
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));            // (what depends on it is computed here, not held in registers all through the kernel)
  constexpr int PER = NBINS / NT;
  int shift = 0;
  while ((((unsigned long long)hi - lo) >> shift) >= (unsigned long long)NBINS) ++shift;
  for (int b = tid; b < NBINS; b += NT) S.hist[b] = 0;
  __syncthreads();
  for (int i = tid; i < n; i += NT) {
    uint32_t v;
    if (val(i, v) && v >= lo && v <= hi) atomicAdd(&S.hist[(v - lo) >> shift], 1u);
  }
  __syncthreads();
  uint32_t loc[PER], sum = 0;
#pragma unroll
  for (int q = 0; q < PER; ++q) { loc[q] = S.hist[tid * PER + q]; sum += loc[q]; }
  int total;
  uint32_t run = (uint32_t)block_excl_scan<NT>((int)sum, S.wave_tmp, total);
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    if (run < need && run + loc[q] >= need) S.sel_bin = tid * PER + q;
    run += loc[q];
  }
  __syncthreads();
  const uint32_t b = S.sel_bin;
  __syncthreads();
  const unsigned long long edge = (unsigned long long)lo + ((unsigned long long)(b + 1) << shift) - 1ull;
  return edge < hi ? (uint32_t)edge : hi;
}

}  // namespace wfst
