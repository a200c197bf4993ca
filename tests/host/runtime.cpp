// The running part of the HIP stand-in (hip/hip_runtime.h): allocations with a
// guard page behind them, and blocks of threads as coroutines.
#include "hip/hip_runtime.h"
#undef asm
#undef volatile

#include <sys/mman.h>

#include <cstdio>
#include <map>
#include <string>
#include <vector>

EmuIndex threadIdx, blockIdx, blockDim, gridDim;

namespace {

[[noreturn]] void stop(const std::string& msg) {
  std::printf("host emulation: %s\n", msg.c_str());
  std::fflush(stdout);
  std::_Exit(3);
}

struct Range {
  size_t n;
  void* map;
  size_t mapped;
};
std::map<const char*, Range> g_ranges;  // by first byte
std::map<std::string, long> g_launches;
std::string g_kernel;
unsigned g_last_grid = 1;
size_t g_live = 0;
double g_trial_ms = 0;

// ---------------------------------------------------------------- coroutines
extern "C" void emu_switch(void** save, void* to);
asm(R"(
.text
.globl emu_switch
emu_switch:
  pushq %rbp
  pushq %rbx
  pushq %r12
  pushq %r13
  pushq %r14
  pushq %r15
  movq %rsp, (%rdi)
  movq %rsi, %rsp
  popq %r15
  popq %r14
  popq %r13
  popq %r12
  popq %rbx
  popq %rbp
  ret
)");

enum State { RUN, WAVE, BLOCK, DONE };
struct Lane {
  char* stack = nullptr;
  void* sp = nullptr;
  State state = DONE;
  EmuIndex tid;
  const void* in = nullptr;
  void* out = nullptr;
  EmuOp op = nullptr;
  int arg = 0;
};
constexpr size_t kStack = 128 << 10;
std::vector<Lane> g_lanes;
Lane* g_cur = nullptr;
void* g_main = nullptr;
const std::function<void()>* g_thread = nullptr;

void yield(State s) {
  Lane* me = g_cur;
  me->state = s;
  emu_switch(&me->sp, g_main);
}
void entry() {
  (*g_thread)();
  yield(DONE);
  stop("a finished thread was resumed");
}
void resume(Lane& l) {
  g_cur = &l;
  l.state = RUN;
  threadIdx = l.tid;
  emu_switch(&g_main, l.sp);
}

// Runs the lanes [l0, l0 + 64) until each has ended or waits for the block.
void run_wave(size_t l0, size_t n) {
  for (;;) {
    int wave = 0, block = 0;
    for (size_t l = l0; l < n; ++l) {
      if (g_lanes[l].state == RUN) resume(g_lanes[l]);
      wave += g_lanes[l].state == WAVE;
      block += g_lanes[l].state == BLOCK;
    }
    if (wave == 0) return;
    if (block > 0) stop("lanes of a wave wait in different places in " + g_kernel);
    void *in[64] = {nullptr}, *out[64] = {nullptr};
    const Lane* first = nullptr;
    for (size_t l = l0; l < n; ++l) {
      const Lane& x = g_lanes[l];
      if (x.state != WAVE) continue;
      if (!first) first = &x;
      if (x.op != first->op || x.arg != first->arg) stop("a wave's lanes are in different operations in " + g_kernel);
      in[l - l0] = const_cast<void*>(x.in);
      out[l - l0] = x.out;
    }
    first->op(in, out, first->arg);
    for (size_t l = l0; l < n; ++l)
      if (g_lanes[l].state == WAVE) g_lanes[l].state = RUN;
  }
}

}  // namespace

void __syncthreads() { yield(BLOCK); }

void emu_wave(const void* in, void* out, EmuOp op, int arg) {
  g_cur->in = in;
  g_cur->out = out;
  g_cur->op = op;
  g_cur->arg = arg;
  yield(WAVE);
}

void emu_launch(const char* name, dim3 grid, dim3 block, const std::function<void()>& thread) {
  std::string k = name;
  k = k.substr(k.find_first_not_of("( "));
  g_kernel = k.substr(0, k.find_first_of("<,) "));
  ++g_launches[g_kernel];
  g_last_grid = grid.x;
  const size_t n = (size_t)block.x * block.y * block.z;
  while (g_lanes.size() < n) {
    Lane l;
    l.stack = (char*)mmap(nullptr, kStack, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    g_lanes.push_back(l);
  }
  g_thread = &thread;
  blockDim = {block.x, block.y, block.z};
  gridDim = {grid.x, grid.y, grid.z};
  for (unsigned bz = 0; bz < grid.z; ++bz)
    for (unsigned by = 0; by < grid.y; ++by)
      for (unsigned bx = 0; bx < grid.x; ++bx) {
        blockIdx = {bx, by, bz};
        for (size_t l = 0; l < n; ++l) {
          Lane& x = g_lanes[l];
          x.tid = {(unsigned)(l % block.x), (unsigned)(l / block.x % block.y), (unsigned)(l / block.x / block.y)};
          void** top = (void**)(x.stack + kStack - 64);
          top[0] = (void*)&entry;  // the return address; above it the callee-saved registers
          x.sp = top - 6;
          x.state = RUN;
        }
        for (;;) {
          size_t waiting = 0;
          for (size_t l = 0; l < n; l += 64) run_wave(l, std::min(n, l + 64));
          for (size_t l = 0; l < n; ++l)
            if (g_lanes[l].state == BLOCK) g_lanes[l].state = RUN, ++waiting;
          if (waiting == 0) break;
        }
      }
}

hipError_t emu_malloc(void** p, size_t n) {
  const size_t page = 4096, body = (n + page - 1) / page * page;
  char* m = (char*)mmap(nullptr, body + page, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
  if (m == MAP_FAILED) return hipErrorOutOfMemory;
  mprotect(m + body, page, PROT_NONE);
  char* at = m + (body - n) / 16 * 16;  // the end at the guard page
  *p = at;
  g_ranges[at] = Range{n, m, body + page};
  g_live += n;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  auto it = g_ranges.find((const char*)p);
  if (it == g_ranges.end()) stop("free of memory that is not allocated");
  g_live -= it->second.n;
  munmap(it->second.map, it->second.mapped);
  g_ranges.erase(it);
  return hipSuccess;
}
hipError_t hipMemGetInfo(size_t* free_b, size_t* total_b) {
  *free_b = *total_b = (size_t)8 << 30;
  return hipSuccess;
}
// What a product's trials measure: all the same, or (emu_trial_ms) the more workgroups, the faster.
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
  *ms = g_trial_ms > 0 ? (float)(g_trial_ms / g_last_grid) : 1.0f;
  return hipSuccess;
}

emu_u4 emu_buffer_load(const EmuBuffer& r, uint32_t v, uint32_t s) {
  if (s > r.size)
    stop("scalar offset " + std::to_string(s) + " beyond a resource of " + std::to_string(r.size) + " bytes in " + g_kernel);
  emu_u4 x = {0, 0, 0, 0};
  if (v >= r.size - s) return x;
  const char* a = r.p + (uint64_t)v + s;
  auto it = g_ranges.upper_bound(a);
  if (it == g_ranges.begin() || (--it, a + 16 > it->first + it->second.n))
    stop("a buffer load outside every allocation in " + g_kernel);
  std::memcpy(&x, a, sizeof(x));
  return x;
}

// For the tests: launches of a kernel since the last reset ("" : all), device memory in use.
extern "C" long emu_launches(const char* name) {
  long n = 0;
  for (auto& kv : g_launches)
    if (!*name || kv.first == name) n += kv.second;
  return n;
}
extern "C" void emu_reset_launches() { g_launches.clear(); }
extern "C" void emu_trial_ms(double of_one_workgroup) { g_trial_ms = of_one_workgroup; }
extern "C" size_t emu_memory_in_use() { return g_live; }
extern "C" void* emu_alloc(size_t n) {
  void* p = nullptr;
  return emu_malloc(&p, n) == hipSuccess ? p : nullptr;
}
