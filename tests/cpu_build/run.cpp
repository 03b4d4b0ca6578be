// Runs a kernel's blocks in turn, a block's threads as fibers that meet at its
// barriers (of the block, and of a wavefront of 64 for the lane exchange).
#include <hip/hip_runtime.h>

#include <dlfcn.h>
#include <ucontext.h>

#include <cstdio>
#include <string>
#include <utility>

dim3 threadIdx, blockIdx, blockDim, gridDim;

namespace cpu {

hipGraph_t capturing = nullptr;
long long calls = 0;
std::vector<std::pair<std::string, unsigned>> launches;   // names and blocks

namespace {
enum State { READY, BLOCK, WAVE, DONE };
constexpr size_t STACK = 1u << 20;
struct Fiber {
  ucontext_t c;
  char* stack = nullptr;
  dim3 id;
  State state = READY;
};
std::vector<Fiber*> fibers;
ucontext_t main_context;
const std::function<void()>* body;
int current, any_or;
double lane[1024];

void wait(State s) {
  Fiber* f = fibers[current];
  f->state = s;
  swapcontext(&f->c, &main_context);
}
void entry() {
  (*body)();
  wait(DONE);
}
void resume(int i) {
  current = i;
  threadIdx = fibers[i]->id;
  swapcontext(&main_context, &fibers[i]->c);
}
// Opens the barrier s of fibers lo .. hi - 1 if every one that is not done waits at it.
bool open(State s, int lo, int hi) {
  bool waiting = false;
  for (int i = lo; i < hi; ++i) {
    if (fibers[i]->state == s) waiting = true;
    else if (fibers[i]->state != DONE) return false;
  }
  if (waiting)
    for (int i = lo; i < hi; ++i)
      if (fibers[i]->state == s) fibers[i]->state = READY;
  return waiting;
}
}  // namespace

void note(void* kernel, unsigned blocks) {
  Dl_info i{};
  dladdr(kernel, &i);
  launches.emplace_back(i.dli_sname ? i.dli_sname : "", blocks);
}

void sync_threads() { wait(BLOCK); }
int sync_or(int v) {
  any_or |= v != 0;
  wait(BLOCK);
  const int r = any_or;
  wait(BLOCK);
  any_or = 0;
  wait(BLOCK);
  return r;
}
double shfl_xor(double v, int mask) {
  const int me = current;
  lane[me] = v;
  wait(WAVE);
  const double r = lane[(me & ~63) + ((me & 63) ^ mask)];
  wait(WAVE);
  return r;
}

void run(dim3 grid, dim3 block, const std::function<void()>& kernel) {
  const int n = block.x * block.y * block.z;
  while ((int)fibers.size() < n) {
    fibers.push_back(new Fiber);
    fibers.back()->stack = (char*)std::malloc(STACK);
  }
  body = &kernel;
  blockDim = block;
  gridDim = grid;
  const unsigned nblocks = grid.x * grid.y * grid.z;
  for (unsigned b = 0; b < nblocks; ++b) {
    blockIdx = dim3(b % grid.x, b / grid.x % grid.y, b / (grid.x * grid.y));
    any_or = 0;
    for (int i = 0; i < n; ++i) {
      Fiber* f = fibers[i];
      getcontext(&f->c);
      f->c.uc_stack.ss_sp = f->stack;
      f->c.uc_stack.ss_size = STACK;
      f->c.uc_link = nullptr;
      f->id = dim3(i % block.x, i / block.x % block.y, i / (block.x * block.y));
      f->state = READY;
      makecontext(&f->c, entry, 0);
    }
    for (;;) {
      bool live = false;
      for (int i = 0; i < n; ++i) {
        if (fibers[i]->state == READY) resume(i);
        live = live || fibers[i]->state != DONE;
      }
      if (!live) break;
      bool opened = false;
      for (int w = 0; w < n; w += 64) opened = open(WAVE, w, w + 64 < n ? w + 64 : n) || opened;
      if (!opened && !open(BLOCK, 0, n)) {
        std::fprintf(stderr, "a barrier that not every thread reaches\n");
        std::abort();
      }
    }
  }
}

}  // namespace cpu

// The calls of exp and log in kernels since the last time.
extern "C" long long cpu_calls() {
  const long long n = cpu::calls;
  cpu::calls = 0;
  return n;
}

// The blocks launched since the last time, of the largest launch (part empty) or
// of all launches of kernels with part in their name.
extern "C" unsigned cpu_blocks(const char* part) {
  unsigned n = 0;
  for (auto& l : cpu::launches)
    if (!*part) n = l.second > n ? l.second : n;
    else if (l.first.find(part) != std::string::npos) n += l.second;
  cpu::launches.clear();
  return n;
}

extern "C" unsigned cpu_largest_grid() { return cpu_blocks(""); }

// Capture as a caller's stream capture would see it.
extern "C" void cpu_capture_begin() { hipStreamBeginCapture(nullptr, hipStreamCaptureModeGlobal); }
extern "C" void* cpu_capture_end() {
  hipGraph_t g;
  hipStreamEndCapture(nullptr, &g);
  return g;
}
extern "C" void cpu_replay(void* g) { hipGraphLaunch((hipGraphExec_t)g, nullptr); }
