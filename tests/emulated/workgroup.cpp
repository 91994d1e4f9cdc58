// Runs workgroups on the CPU (see hip/hip_runtime.h).  Between two barriers the wavefronts of a workgroup run one after
// the other, each as far as it gets - the first one first, or, with EMULATED_ORDER set, in an order drawn anew every time -
// so that what a wavefront relies on without a barrier shows.
#include <hip/hip_runtime.h>
#include <sched.h>
#include <stdio.h>
#include <sys/mman.h>
#include <map>
#include <mutex>
#include <thread>
#include <vector>

thread_local uint3 threadIdx, blockIdx, blockDim, gridDim;

// Saves the callee's registers and the stack pointer, and goes on where another stack was left.
extern "C" void switch_stack(void **save, void *load);
asm(R"(
.text
.globl switch_stack
switch_stack:
  pushq %rbp; pushq %rbx; pushq %r12; pushq %r13; pushq %r14; pushq %r15
  movq %rsp, (%rdi)
  movq %rsi, %rsp
  popq %r15; popq %r14; popq %r13; popq %r12; popq %rbx; popq %rbp
  ret
)");

namespace {

enum { READY, WAITS, OVER };
constexpr size_t STACK = 128 << 10;
struct Thread { void *sp; int state, op; uint64_t v, arg, old, result; };
struct Stacks {
  char *base = (char *)mmap(nullptr, STACK * 1024, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
  ~Stacks() { munmap(base, STACK * 1024); }
};
struct Workgroup { std::vector<Thread> t; void *scheduler; int current; const std::function<void()> *kernel; };
thread_local Workgroup W;

void entry() {
  (*W.kernel)();
  Thread &me = W.t[W.current];
  me.state = OVER;
  for (;;) switch_stack(&me.sp, W.scheduler);
}

[[noreturn]] void give_up(const char *what, int wave) {
  fprintf(stderr, "workgroup %u, wavefront %d: %s\n", blockIdx.x, wave, what);
  abort();
}

// Lanes in a branch: each gets the result of those that wait for the same in the same place.
void perform_here(int a, int e) {
  for (int i = a; i < e; ++i) {
    Thread &t = W.t[i];
    if (t.state != WAITS || t.op < OP_BALLOT_HERE) continue;
    auto beside = [&](int k) { return W.t[k].state == WAITS && W.t[k].op == t.op && W.t[k].old == t.old; };
    t.result = 0;
    if (t.op == OP_READLANE_HERE) {
      if (a + (int)t.arg >= e || !beside(a + (int)t.arg)) give_up("a lane is read that is not here", a / 64);
      t.result = W.t[a + (int)t.arg].v;
    } else {
      for (int k = a; k < e; ++k) if (beside(k) && W.t[k].v) t.result |= 1ull << (k - a);
    }
  }
  for (int i = a; i < e; ++i) if (W.t[i].state == WAITS && W.t[i].op >= OP_BALLOT_HERE) W.t[i].state = READY;
}

// All threads of the wavefront [a, e) that are not over wait for `op`: every one gets its result.
void perform(int op, int a, int e) {
  uint64_t mask = 0, v[64] = {};
  int first = -1;
  for (int i = a; i < e; ++i) if (W.t[i].state == WAITS) {
    v[i - a] = W.t[i].v;
    if (first < 0) first = i - a;
    if (W.t[i].v) mask |= 1ull << (i - a);
  }
  for (int i = a; i < e; ++i) if (W.t[i].state == WAITS) {
    Thread &t = W.t[i];
    const int l = i - a, n = (int)t.arg;
    switch (op) {
      case OP_BALLOT: t.result = mask; break;
      case OP_READLANE: t.result = v[n & 63]; break;
      case OP_READFIRST: t.result = v[first]; break;
      case OP_DPP: t.result = (l & 15) >= (n & 15) ? v[l - (n & 15)] : t.old; break;        // (row_shr, the only control in use)
      case OP_UP: t.result = l >= n ? v[l - n] : v[l]; break;
      case OP_XOR: t.result = v[l ^ n]; break;
    }
    t.state = READY;
  }
}

void run_workgroup(uint32_t index, dim3 grid, dim3 block, const std::function<void()> &kernel) {
  static thread_local Stacks own;
  char *const stacks = own.base;
  static thread_local uint64_t drawn = 88172645463325252ull;
  const bool any_order = getenv("EMULATED_ORDER") != nullptr;
  blockIdx = uint3{index % grid.x, index / grid.x, 0}; blockDim = uint3{block.x, 1, 1}; gridDim = uint3{grid.x, grid.y, 1};
  const int n = (int)block.x, waves = (n + 63) / 64;
  W.kernel = &kernel;
  W.t.assign((size_t)n, Thread{});
  for (int i = 0; i < n; ++i) {
    void **s = (void **)(stacks + STACK * (size_t)(i + 1));
    *--s = nullptr; *--s = (void *)entry;
    for (int k = 0; k < 6; ++k) *--s = nullptr;
    W.t[i].sp = s;
  }
  std::vector<int> order((size_t)waves);
  for (int w = 0; w < waves; ++w) order[w] = w;
  for (int left = n; left > 0;) {
    bool went_on = false, sleeps = false;
    int at_barrier = 0;
    for (int w = waves - 1; any_order && w > 0; --w) {
      drawn ^= drawn << 13; drawn ^= drawn >> 7; drawn ^= drawn << 17;
      std::swap(order[w], order[drawn % (uint64_t)(w + 1)]);
    }
    for (const int w : order) {
      const int a = w * 64, e = std::min(n, a + 64);
      for (bool more = true; more;) {
        for (int i = a; i < e; ++i) if (W.t[i].state == READY) {
          W.current = i; threadIdx = uint3{(uint32_t)i, 0, 0};
          switch_stack(&W.scheduler, W.t[i].sp);
          went_on = true;
          if (W.t[i].state == OVER) --left;
        }
        int op = 0;
        bool slept = false, here = false;
        for (int i = a; i < e; ++i) here |= W.t[i].state == WAITS && W.t[i].op >= OP_BALLOT_HERE;
        if (here) { perform_here(a, e); continue; }
        for (int i = a; i < e; ++i) if (W.t[i].state == WAITS) {
          if (W.t[i].op == OP_SLEEP) { W.t[i].state = READY; slept = true; continue; }
          if (op != 0 && op != W.t[i].op) give_up("its threads wait for different things", w);
          op = W.t[i].op;
        }
        sleeps |= slept;
        more = !slept && op != 0 && op != OP_BARRIER;
        if (more) perform(op, a, e);
      }
      for (int i = a; i < e; ++i) at_barrier += W.t[i].state == WAITS && W.t[i].op == OP_BARRIER;
    }
    if (left > 0 && at_barrier == left) {
      for (Thread &t : W.t) if (t.state == WAITS) t.state = READY;
    } else if (sleeps) {
      sched_yield();
    } else if (!went_on && left > 0) {
      give_up("some wait at a barrier that the others do not come to", 0);
    }
  }
}

std::map<void *, std::pair<char *, size_t>> allocated;
std::mutex allocating;

}  // namespace

uint64_t together(int op, uint64_t v, uint64_t arg, uint64_t old) {
  Thread &me = W.t[W.current];
  me.op = op; me.v = v; me.arg = arg; me.old = old; me.state = WAITS;
  switch_stack(&me.sp, W.scheduler);
  return me.result;
}

void run_grid(dim3 grid, dim3 block, bool at_once, const std::function<void()> &kernel) {
  const uint32_t n = grid.x * grid.y;
  uint32_t next = 0;
  std::vector<std::thread> workers;
  for (uint32_t k = 0; k < (at_once ? n : std::min(n, 8u)); ++k)
    workers.emplace_back([&]() {
      for (uint32_t i; (i = __atomic_fetch_add(&next, 1u, __ATOMIC_SEQ_CST)) < n;) run_workgroup(i, grid, block, kernel);
    });
  for (std::thread &w : workers) w.join();
}

hipError_t hipMalloc(void **p, size_t n) {
  const size_t page = 4096, body = (n + 15) & ~(size_t)15, length = (body + page - 1) / page * page + 2 * page;
  char *m = (char *)mmap(nullptr, length, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
  if (m == MAP_FAILED) return 2;
  mprotect(m, page, PROT_NONE);
  mprotect(m + length - page, page, PROT_NONE);
  *p = getenv("EMULATED_ORDER") ? m + page : m + length - page - body;
  if (n <= (size_t)32 << 20) memset(*p, 0xCD, body);            // (nobody may count on zeros)
  std::lock_guard<std::mutex> lock(allocating);
  allocated[*p] = {m, length};
  return 0;
}
hipError_t hipFree(void *p) {
  if (!p) return 0;
  std::lock_guard<std::mutex> lock(allocating);
  const auto it = allocated.find(p);
  if (it == allocated.end()) abort();
  munmap(it->second.first, it->second.second);
  allocated.erase(it);
  return 0;
}
extern "C" void *emulated_alloc(size_t n) { void *p = nullptr; return hipMalloc(&p, n) == 0 ? p : nullptr; }
