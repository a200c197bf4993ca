// A stand-in for the HIP runtime and the device builtins that the library's
// sources use, so that they compile and run on the CPU: launches run their
// threads one block after another, the lanes of a wave meet at its cross-lane
// operations (runtime.cpp), and a buffer load is checked against its resource
// and against the allocations.  Only what the sources use is here.
#pragma once

#include <cmath>
#include <cstddef>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <tuple>

// ---------------------------------------------------------------- host API
enum hipError_t { hipSuccess = 0, hipErrorOutOfMemory = 2, hipErrorNotSupported = 801 };
enum hipMemcpyKind { hipMemcpyHostToDevice = 1, hipMemcpyDeviceToHost = 2, hipMemcpyDeviceToDevice = 3 };
enum hipStreamCaptureMode { hipStreamCaptureModeThreadLocal = 1 };
enum { hipStreamNonBlocking = 1, hipEventDisableTiming = 2 };
typedef struct ihipStream_t* hipStream_t;
typedef struct ihipEvent_t* hipEvent_t;
typedef struct ihipGraph* hipGraph_t;
typedef struct hipGraphExec* hipGraphExec_t;
struct dim3 {
  unsigned x, y, z;
  dim3(unsigned a = 1, unsigned b = 1, unsigned c = 1) : x(a), y(b), z(c) {}
};

hipError_t emu_malloc(void** p, size_t n);
template <class T>
hipError_t hipMalloc(T** p, size_t n) {
  return emu_malloc((void**)p, n);
}
hipError_t hipFree(void* p);
hipError_t hipMemGetInfo(size_t* free_b, size_t* total_b);
hipError_t hipEventElapsedTime(float* ms, hipEvent_t a, hipEvent_t b);
inline hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { return std::memmove(d, s, n), hipSuccess; }
inline hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
  return std::memmove(d, s, n), hipSuccess;
}
inline hipError_t hipMemset(void* d, int v, size_t n) { return std::memset(d, v, n), hipSuccess; }
inline hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) { return std::memset(d, v, n), hipSuccess; }
template <class T>
hipError_t emu_handle(T* p) {
  static uintptr_t next = 16;
  *p = (T)(next += 16);
  return hipSuccess;
}
inline hipError_t hipStreamCreate(hipStream_t* s) { return emu_handle(s); }
inline hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { return emu_handle(s); }
inline hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
inline hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
inline hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
inline hipError_t hipDeviceSynchronize() { return hipSuccess; }
inline hipError_t hipEventCreate(hipEvent_t* e) { return emu_handle(e); }
inline hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return emu_handle(e); }
inline hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
inline hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
inline hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
inline hipError_t hipGetLastError() { return hipSuccess; }
inline const char* hipGetErrorString(hipError_t) { return "host emulation"; }
inline hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
inline hipError_t hipGetSymbolAddress(void** p, void* s) { return *p = s, hipSuccess; }
#define HIP_SYMBOL(x) ((void*)(x))
inline hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipErrorNotSupported; }
inline hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t*) { return hipErrorNotSupported; }
inline hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
inline hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
inline hipError_t hipGraphInstantiate(hipGraphExec_t*, hipGraph_t, void*, void*, size_t) { return hipErrorNotSupported; }
inline hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipErrorNotSupported; }

// ---------------------------------------------------------------- launches
void emu_launch(const char* name, dim3 grid, dim3 block, const std::function<void()>& thread);
template <class... P, class... A>
void emu_start(const char* name, void (*kernel)(P...), dim3 grid, dim3 block, A... args) {
  const std::tuple<std::decay_t<P>...> a(args...);
  emu_launch(name, grid, block, [&]() { std::apply(kernel, a); });
}
#define hipLaunchKernelGGL(kernel, grid, block, shared, stream, ...) \
  ((void)(stream), emu_start(#kernel, kernel, dim3(grid), dim3(block), __VA_ARGS__))

// ---------------------------------------------------------------- device side
#define __global__
#define __device__
#define __host__
#define __constant__
#define __shared__ static
#define __forceinline__ inline
#define __launch_bounds__(...)
#define __align__(n) __attribute__((aligned(n)))
// register constraints and scheduling fences have no meaning here: asm volatile("" : ...) is dropped
#define asm
#define volatile(...)
#define __builtin_amdgcn_sched_barrier(x)

struct int4 {
  int x, y, z, w;
};
struct EmuIndex {
  unsigned x, y, z;
};
extern EmuIndex threadIdx, blockIdx, blockDim, gridDim;

using std::isfinite;
inline int min(int a, int b) { return a < b ? a : b; }
inline int max(int a, int b) { return a > b ? a : b; }
inline uint32_t __umulhi(uint32_t a, uint32_t b) { return (uint32_t)((uint64_t)a * b >> 32); }
inline double unsafeAtomicAdd(double* p, double x) { return *p += x; }
inline int atomicCAS(int* p, int expect, int x) {
  const int old = *p;
  if (old == expect) *p = x;
  return old;
}

void __syncthreads();
// A cross-lane operation: called once all running lanes of the wave are in it,
// with their inputs and results (null for lanes that have ended).
typedef void (*EmuOp)(void* const* in, void* const* out, int arg);
void emu_wave(const void* in, void* out, EmuOp op, int arg);
template <class T>
T __shfl_xor(T x, int mask) {
  T y;
  emu_wave(
      &x, &y,
      [](void* const* in, void* const* out, int m) {
        for (int l = 0; l < 64; ++l)
          if (out[l]) *(T*)out[l] = *(const T*)in[l ^ m];
      },
      mask);
  return y;
}
inline int emu_readfirstlane(int x) {
  int y;
  emu_wave(
      &x, &y,
      [](void* const* in, void* const* out, int) {
        int first = 0;
        while (!in[first]) ++first;
        for (int l = 0; l < 64; ++l)
          if (out[l]) *(int*)out[l] = *(const int*)in[first];
      },
      0);
  return y;
}
#define __builtin_amdgcn_readfirstlane(x) emu_readfirstlane(x)

// D = A B + C of a wave: lane l holds A[l%16][KL*(l/16) + 0..KL-1], B likewise by
// columns; result register r is D[4r + l/16][l%16] (INTERLEAVED) or D[4(l/16) + r][l%16].
template <class E, class D, int KL, bool INTERLEAVED>
D emu_mfma(E a, E b, D c) {
  struct In {
    E a, b;
    D c;
  } x{a, b, c};
  D y;
  emu_wave(
      &x, &y,
      [](void* const* in, void* const* out, int) {
        typedef std::decay_t<decltype(D()[0])> T;
        constexpr int K = 4 * KL;
        T A[16][K], B[K][16];
        auto get = [](const E& v, int e) {
          if constexpr (KL == 1)
            return v;
          else
            return (T)v[e];
        };
        for (int l = 0; l < 64; ++l)
          for (int e = 0; e < KL; ++e) {
            A[l % 16][l / 16 * KL + e] = get(((const In*)in[l])->a, e);
            B[l / 16 * KL + e][l % 16] = get(((const In*)in[l])->b, e);
          }
        for (int l = 0; l < 64; ++l) {
          D d = ((const In*)in[l])->c;
          for (int r = 0; r < 4; ++r) {
            const int m = INTERLEAVED ? 4 * r + l / 16 : 4 * (l / 16) + r;
            T t = d[r];
            for (int k = 0; k < K; ++k) t += A[m][k] * B[k][l % 16];
            d[r] = t;
          }
          std::memcpy(out[l], &d, sizeof(d));
        }
      },
      0);
  return y;
}
typedef double emu_d4 __attribute__((ext_vector_type(4)));
typedef float emu_f4 __attribute__((ext_vector_type(4)));
#define __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, x, y, z) emu_mfma<double, emu_d4, 1, true>(a, b, c)
#define __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, x, y, z) emu_mfma<float, emu_f4, 1, false>(a, b, c)
#define __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, x, y, z) emu_mfma<decltype(a), emu_f4, 8, false>(a, b, c)

// A raw buffer: a load at lane offset v and scalar offset s reads zero where
// v >= size - s, formed in 32 bits without a sign, so that s must not exceed
// the size; in range, it must lie in an allocation.
struct EmuBuffer {
  const char* p;
  uint32_t size;
};
typedef uint32_t emu_u4 __attribute__((ext_vector_type(4)));
emu_u4 emu_buffer_load(const EmuBuffer& r, uint32_t v, uint32_t s);
#define __amdgpu_buffer_rsrc_t EmuBuffer
#define __builtin_amdgcn_make_buffer_rsrc(p, stride, n, flags) (EmuBuffer{(const char*)(p), (uint32_t)(n)})
#define __builtin_amdgcn_raw_buffer_load_b128(r, v, s, aux) emu_buffer_load(r, (uint32_t)(v), (uint32_t)(s))
