// Host stand-in for the HIP runtime, for running the line and tile kernels on
// the CPU (tests/test_host_kernels.py): a launch runs its workgroups one after
// the other, the threads of a workgroup as fibers that switch only at barriers.
//
// Between two barriers each wave runs to the end before the next one starts,
// in ascending or (emu::reversed) descending order of workgroups, waves and
// lanes.  A kernel whose results differ between the two orders reads memory or
// LDS without the barrier that would order it after the write.  LDS holds NaN before a
// workgroup starts and guard words after the launch's LDS bytes.
#pragma once
#include <ucontext.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#define __global__
#define __host__
#define __device__
#define __forceinline__ inline
#define __launch_bounds__(...)
#define __shared__ static
#define EMU_ASM(...)

struct alignas(8) float2 {
  float x, y;
};
inline float2 make_float2(float x, float y) { return {x, y}; }
struct dim3 {
  unsigned x, y, z;
  dim3(unsigned x_ = 1, unsigned y_ = 1, unsigned z_ = 1) : x(x_), y(y_), z(z_) {}
};

template <class T>
inline T min(T a, T b) { return a < b ? a : b; }
template <class T>
inline T max(T a, T b) { return a > b ? a : b; }
inline unsigned __umulhi(unsigned a, unsigned b) { return (unsigned)(((unsigned long long)a * b) >> 32); }
inline unsigned __float_as_uint(float f) {
  unsigned u;
  std::memcpy(&u, &f, 4);
  return u;
}
inline float __uint_as_float(unsigned u) {
  float f;
  std::memcpy(&f, &u, 4);
  return f;
}
typedef _Float16 __half;
inline __half __ushort_as_half(unsigned short u) {
  __half h;
  std::memcpy(&h, &u, 2);
  return h;
}
inline unsigned short __half_as_ushort(__half h) {
  unsigned short u;
  std::memcpy(&u, &h, 2);
  return u;
}
inline float __half2float(__half h) { return (float)h; }
inline __half __float2half_rn(float f) { return (__half)f; }
#define __builtin_amdgcn_sqrtf sqrtf
#define __builtin_amdgcn_logf log2f
#define __builtin_amdgcn_exp2f exp2f

typedef void* hipStream_t;
typedef void* hipEvent_t;
typedef int hipError_t;
enum { hipSuccess = 0, hipDeviceAttributeMultiprocessorCount = 1, hipFuncAttributeMaxDynamicSharedMemorySize = 2 };
inline hipError_t hipGetLastError() { return hipSuccess; }
inline const char* hipGetErrorString(hipError_t) { return ""; }
inline hipError_t hipEventCreate(hipEvent_t*) { return hipSuccess; }
inline hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
inline hipError_t hipEventElapsedTime(float* t, hipEvent_t, hipEvent_t) { return *t = 0.f, hipSuccess; }
inline hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
inline hipError_t hipFuncSetAttribute(const void*, int, int) { return hipSuccess; }

extern dim3 threadIdx, blockIdx, blockDim, gridDim;

namespace os3d {
extern float2 lds[];
}

namespace emu {

constexpr int kMaxThreads = 1024;
constexpr size_t kLds = 160 * 1024, kGuard = 16 * 1024, kStack = 64 * 1024;
constexpr unsigned char kNaN = 0xff, kCanary = 0xa5;
extern int compute_units;  // what the device reports
extern bool reversed;      // order of workgroups, waves and lanes
enum Stop { kRunning, kBarrier, kWave, kDone };

struct Fibers {
  ucontext_t main, ctx[kMaxThreads];
  std::vector<char> stacks;
  Stop stop[kMaxThreads];
  float lane[kMaxThreads];  // values of a wave exchange
  int cur = 0;
  void (*call)(void*) = nullptr;
  void* arg = nullptr;
  Fibers() : stacks(kMaxThreads * kStack) {}
};
extern Fibers fibers;

[[noreturn]] inline void fail(const char* what) {
  std::printf("emulation: %s\n", what);
  std::fflush(stdout);
  std::exit(3);
}

inline void yield(Stop s) {
  const int t = fibers.cur;
  fibers.stop[t] = s;
  swapcontext(&fibers.ctx[t], &fibers.main);
}

inline void entry() {
  fibers.call(fibers.arg);
  fibers.stop[fibers.cur] = kDone;
}

inline void resume(int t) {
  fibers.cur = t;
  threadIdx = dim3((unsigned)t, 0, 0);
  swapcontext(&fibers.main, &fibers.ctx[t]);
}

// The lanes of a wave to its next barrier or its end.
inline Stop run_wave(int w, int n) {
  const int lo = w * 64, hi = std::min(n, lo + 64);
  for (;;) {
    for (int i = lo; i < hi; ++i) resume(reversed ? lo + hi - 1 - i : i);
    for (int i = lo; i < hi; ++i)
      if (fibers.stop[i] != fibers.stop[lo]) fail("the lanes of a wave stop at different places");
    if (fibers.stop[lo] != kWave) return fibers.stop[lo];
  }
}

inline void run_workgroup(int n, size_t lds) {
  char* base = (char*)os3d::lds;
  std::memset(base, kNaN, lds);
  std::memset(base + lds, kCanary, kGuard);
  for (int t = 0; t < n; ++t) {
    getcontext(&fibers.ctx[t]);
    fibers.ctx[t].uc_stack.ss_sp = fibers.stacks.data() + (size_t)t * kStack;
    fibers.ctx[t].uc_stack.ss_size = kStack;
    fibers.ctx[t].uc_link = &fibers.main;
    makecontext(&fibers.ctx[t], entry, 0);
  }
  const int waves = (n + 63) / 64;
  for (bool done = false; !done;) {
    Stop all = kRunning;
    for (int i = 0; i < waves; ++i) {
      const Stop s = run_wave(reversed ? waves - 1 - i : i, n);
      if (all != kRunning && s != all) fail("a barrier that some waves do not reach");
      all = s;
    }
    done = all == kDone;
  }
  for (size_t i = 0; i < kGuard; ++i)
    if ((unsigned char)base[lds + i] != kCanary) fail("a write past the LDS of the launch");
}

template <class F>
void launch(dim3 grid, dim3 block, size_t lds, F body) {
  if (block.x > kMaxThreads || lds > kLds || !block.x || !grid.x || !grid.y) fail("launch limits");
  gridDim = grid;
  blockDim = block;
  fibers.arg = &body;
  fibers.call = [](void* p) { (*(F*)p)(); };
  const long long n = (long long)grid.x * grid.y;
  for (long long i = 0; i < n; ++i) {
    const long long g = reversed ? n - 1 - i : i;
    blockIdx = dim3((unsigned)(g % grid.x), (unsigned)(g / grid.x), 0);
    run_workgroup((int)block.x, lds);
  }
}

}  // namespace emu

inline hipError_t hipDeviceGetAttribute(int* v, int, int) { return *v = emu::compute_units, hipSuccess; }
inline void __syncthreads() { emu::yield(emu::kBarrier); }
inline float __shfl_xor(float v, int o) {
  const int t = emu::fibers.cur;
  emu::fibers.lane[t] = v;
  emu::yield(emu::kWave);
  const float r = emu::fibers.lane[t ^ o];
  emu::yield(emu::kWave);
  return r;
}
#define hipLaunchKernelGGL(kernel, grid, block, lds, st, ...) \
  emu::launch(grid, block, lds, [&]() { kernel(__VA_ARGS__); })
#define hipExtLaunchKernelGGL(kernel, grid, block, lds, st, e0, e1, flags, ...) \
  emu::launch(grid, block, lds, [&]() { kernel(__VA_ARGS__); })
