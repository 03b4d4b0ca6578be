// The part of HIP that the library uses, on the CPU: tests compile its sources
// with this header in HIP's place and run the kernels here, a block's threads as
// fibers and the blocks in turn.  Device memory is malloc's, filled with NaNs.
#pragma once
#include <math.h>

#include <cmath>
#include <cstddef>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <tuple>
#include <type_traits>
#include <vector>

#define __global__
#define __device__
#define __host__
#define __forceinline__ inline
#define __shared__ static
#define __launch_bounds__(...)
#define __align__(n) __attribute__((aligned(n)))

struct int3 { int x, y, z; };
struct dim3 {
  unsigned x, y, z;
  dim3(unsigned a = 1, unsigned b = 1, unsigned c = 1) : x(a), y(b), z(c) {}
};
struct alignas(16) double2 { double x, y; };
extern dim3 threadIdx, blockIdx, blockDim, gridDim;

typedef int hipError_t;
enum { hipSuccess = 0, hipErrorInvalidValue = 1, hipErrorOutOfMemory = 2 };
typedef struct cpu_stream* hipStream_t;
typedef struct cpu_event* hipEvent_t;
struct cpu_graph { std::vector<std::function<void()>> nodes; };
typedef cpu_graph* hipGraph_t;
typedef cpu_graph* hipGraphExec_t;
enum hipMemcpyKind { hipMemcpyHostToDevice, hipMemcpyDeviceToHost, hipMemcpyDeviceToDevice };
enum hipStreamCaptureStatus { hipStreamCaptureStatusNone, hipStreamCaptureStatusActive };
enum hipStreamCaptureMode { hipStreamCaptureModeGlobal, hipStreamCaptureModeThreadLocal };
enum hipDeviceAttribute_t { hipDeviceAttributeMultiprocessorCount };
enum { hipEventDisableTiming = 2, hipStreamNonBlocking = 1 };

namespace cpu {
extern hipGraph_t capturing;
void sync_threads();
int sync_or(int v);
double shfl_xor(double v, int mask);
void run(dim3 grid, dim3 block, const std::function<void()>& kernel);
void note(void* kernel, unsigned blocks);
inline void submit(std::function<void()> f) {
  if (capturing) capturing->nodes.push_back(std::move(f));
  else f();
}
template <class... P, class... A>
void launch(dim3 grid, dim3 block, void (*kernel)(P...), A... args) {
  std::tuple<std::decay_t<P>...> t(args...);   // by value at the launch, as a graph's node keeps them
  note((void*)kernel, grid.x * grid.y * grid.z);
  submit([=] { run(grid, block, [=] { std::apply(kernel, t); }); });
}
}  // namespace cpu
#define hipLaunchKernelGGL(K, G, B, LDS, STREAM, ...) cpu::launch(dim3(G), dim3(B), K, __VA_ARGS__)

inline void __syncthreads() { cpu::sync_threads(); }
inline int __syncthreads_or(int v) { return cpu::sync_or(v); }
inline double __shfl_xor(double v, int mask, int = 64) { return cpu::shfl_xor(v, mask); }
// lane by lane: a lane for which p is false changes nothing in such a branch
inline int __any(int p) { return p; }
inline int __double2hiint(double x) {
  int64_t b;
  std::memcpy(&b, &x, 8);
  return (int)(b >> 32);
}
inline double __hiloint2double(int hi, int lo) {
  const int64_t b = (int64_t)hi << 32 | (uint32_t)lo;
  double x;
  std::memcpy(&x, &b, 8);
  return x;
}
// the hardware's estimates: about half the digits
inline double cpu_estimate(double y) { return std::isnormal(y) ? y * (1 + 1e-8) : y; }
#define __builtin_amdgcn_rcp(x) cpu_estimate(1.0 / (x))
#define __builtin_amdgcn_rsq(x) cpu_estimate(1.0 / std::sqrt(x))
#define __builtin_amdgcn_readfirstlane(x) (x)
inline unsigned min(unsigned a, unsigned b) { return a < b ? a : b; }
template <class T> T atomicAdd(T* p, T v) { T o = *p; *p += v; return o; }
template <class T, class S> T atomicOr(T* p, S v) { T o = *p; *p |= (T)v; return o; }

template <class T> hipError_t hipMalloc(T** p, size_t n) {
  *p = (T*)std::malloc(n ? n : 1);
  std::memset((void*)*p, 0xff, n);
  return hipSuccess;
}
inline hipError_t hipFree(void* p) { std::free(p); return hipSuccess; }
inline hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
inline hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
  cpu::submit([=] { std::memcpy(d, s, n); });
  return hipSuccess;
}
inline hipError_t hipMemset(void* d, int v, size_t n) { std::memset(d, v, n); return hipSuccess; }
inline const char* hipGetErrorString(hipError_t) { return "error"; }
inline hipError_t hipGetLastError() { return hipSuccess; }
inline hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
inline hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
inline hipError_t hipDeviceSynchronize() { return hipSuccess; }
inline hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
inline hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
inline hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = nullptr; return hipSuccess; }
inline hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
inline hipError_t hipEventCreate(hipEvent_t* e) { *e = nullptr; return hipSuccess; }
inline hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = nullptr; return hipSuccess; }
inline hipError_t hipEventRecord(hipEvent_t, hipStream_t = nullptr) { return hipSuccess; }
inline hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
inline hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
inline hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 1.0f; return hipSuccess; }
inline hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) {
  *s = cpu::capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
inline hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { cpu::capturing = new cpu_graph; return hipSuccess; }
inline hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) {
  *g = cpu::capturing;
  cpu::capturing = nullptr;
  return hipSuccess;
}
inline hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t g, void*, void*, size_t) { *e = new cpu_graph(*g); return hipSuccess; }
inline hipError_t hipGraphLaunch(hipGraphExec_t e, hipStream_t) {
  for (auto& n : e->nodes) n();
  return hipSuccess;
}
inline hipError_t hipGraphDestroy(hipGraph_t g) { delete g; return hipSuccess; }
inline hipError_t hipGraphExecDestroy(hipGraphExec_t g) { delete g; return hipSuccess; }
#define HIP_SYMBOL(x) x
inline hipError_t hipGetSymbolAddress(void** p, const void* s) { *p = const_cast<void*>(s); return hipSuccess; }

// In the kernels' files: the calls of exp and log are counted.
#ifdef CPU_COUNT_CALLS
namespace cpu { extern long long calls; }
inline double cpu_exp(double x) { ++cpu::calls; return exp(x); }
inline double cpu_log(double x) { ++cpu::calls; return log(x); }
#define exp cpu_exp
#define log cpu_log
#endif
