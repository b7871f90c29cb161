// Internal helpers shared by the gfx950 kernels and the host orchestrator.
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_bf16.h>
#include <stdint.h>
#include <math.h>

#include "../../include/sb.h"

namespace sb {

constexpr double kLog2Pi = 1.8378770664093454835606594728112;
constexpr int kWave = 64;
constexpr int kMaxHist = 8;   // largest L-BFGS memory held in registers
constexpr int kMaxComp = 16;  // largest mixture (responsibilities held per row in registers)
constexpr int kMaxMem = 32;   // largest L-BFGS memory (beyond kMaxHist the history is
                              // streamed from memory in each loop of the recursion)

typedef uint16_t bf16_t;  // raw bit pattern; converted with round-to-nearest-even

__host__ __device__ inline bf16_t f32_to_bf16(float f) {
  union { float f; uint32_t u; } v;
  v.f = f;
  uint32_t u = v.u;
  if ((u & 0x7f800000u) == 0x7f800000u) {  // inf / nan: keep class
    uint16_t h = (uint16_t)(u >> 16);
    if (u & 0x007fffffu) h |= 0x0040u;
    return h;
  }
  u += 0x7fffu + ((u >> 16) & 1u);
  return (bf16_t)(u >> 16);
}

__host__ __device__ inline float bf16_to_f32(bf16_t h) {
  union { uint32_t u; float f; } v;
  v.u = ((uint32_t)h) << 16;
  return v.f;
}

// ---------------------------------------------------------------- reductions
// Butterfly partners without an LDS trip (all 64 lanes active).  Lanes 32 and
// 16 apart meet through the row swaps; 8, 4, 2 and 1 apart through DPP row
// rotations and quad permutations.  The rotation by four meets lane l - 4
// instead of lane l ^ 4, which holds the same value once the step of eight is
// done.  Every lane adds the pairs of a __shfl_xor butterfly, so results are
// the same bits; a step costs a few VALU cycles instead of the LDS round trip
// (twice, for a double) of the shuffle.  It bounds the L-BFGS step, whose
// recursion is a chain of such sums: whole path at d = 1024, K = 8 102.5 ->
// 99.2 ms, d = 64, K = 4 in FP64 3.91 -> 3.70 ms.
template <int CTRL>
__device__ inline int dpp_mov(int v) {
  return __builtin_amdgcn_mov_dpp(v, CTRL, 0xf, 0xf, true);
}
constexpr int kDppRor8 = 0x128, kDppRor4 = 0x124, kDppXor2 = 0x4e, kDppXor1 = 0xb1,
              kDppHalfMirror = 0x141;
template <int CTRL>
__device__ inline float dpp_val(float v) {
  return __int_as_float(dpp_mov<CTRL>(__float_as_int(v)));
}
template <int CTRL>
__device__ inline double dpp_val(double v) {
  return __hiloint2double(dpp_mov<CTRL>(__double2hiint(v)), dpp_mov<CTRL>(__double2loint(v)));
}
template <int ROW>  // a, b: the values of this lane's row pair (ROW lanes apart)
__device__ inline void row_pair(int v, int &a, int &b) {
  if constexpr (ROW == 32) {
    const auto r = __builtin_amdgcn_permlane32_swap((unsigned)v, (unsigned)v, false, false);
    a = (int)r[0];
    b = (int)r[1];
  } else {
    const auto r = __builtin_amdgcn_permlane16_swap((unsigned)v, (unsigned)v, false, false);
    a = (int)r[0];
    b = (int)r[1];
  }
}
template <int ROW>
__device__ inline void row_pair(float v, float &a, float &b) {
  int x, y;
  row_pair<ROW>(__float_as_int(v), x, y);
  a = __int_as_float(x);
  b = __int_as_float(y);
}
template <int ROW>
__device__ inline void row_pair(double v, double &a, double &b) {
  int xl, yl, xh, yh;
  row_pair<ROW>(__double2loint(v), xl, yl);
  row_pair<ROW>(__double2hiint(v), xh, yh);
  a = __hiloint2double(xh, xl);
  b = __hiloint2double(yh, yl);
}
// Sum over the wave, in the order of a butterfly from 32 lanes down to 1.
template <typename T>
__device__ inline T wave_sum(T v) {
  if constexpr (__is_floating_point(T)) {
    T a, b;
    row_pair<32>(v, a, b);
    v = a + b;
    row_pair<16>(v, a, b);
    v = a + b;
    v += dpp_val<kDppRor8>(v);
    v += dpp_val<kDppRor4>(v);
    v += dpp_val<kDppXor2>(v);
    v += dpp_val<kDppXor1>(v);
  } else {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  }
  return v;
}
// Max over the wave; NaN inputs are ignored (fmax semantics).
template <typename T>
__device__ inline T wave_max(T v) {
  T a, b;
  row_pair<32>(v, a, b);
  v = fmax(a, b);
  row_pair<16>(v, a, b);
  v = fmax(a, b);
  v = fmax(v, dpp_val<kDppRor8>(v));
  v = fmax(v, dpp_val<kDppRor4>(v));
  v = fmax(v, dpp_val<kDppXor2>(v));
  v = fmax(v, dpp_val<kDppXor1>(v));
  return v;
}

// Sum over a block of TPB threads (TPB a multiple of 64); every thread gets
// the total.  `red` is LDS scratch of >= TPB/64 elements per value.  Fixed
// order: waves reduce by butterfly, then wave totals are added in order.
template <int TPB, typename T>
__device__ inline T block_sum(T v, T *red) {
  v = wave_sum(v);
  if constexpr (TPB == 64) {
    return v;
  } else {
    const int w = threadIdx.x / 64, l = threadIdx.x % 64;
    __syncthreads();
    if (l == 0) red[w] = v;
    __syncthreads();
    T t = red[0];
#pragma unroll
    for (int i = 1; i < TPB / 64; ++i) t += red[i];
    return t;
  }
}

// Several sums at once (N values), same ordering rule.
template <int TPB, int N, typename T>
__device__ inline void block_sum_n(T (&v)[N], T *red) {
#pragma unroll
  for (int j = 0; j < N; ++j) v[j] = wave_sum(v[j]);
  if constexpr (TPB > 64) {
    const int w = threadIdx.x / 64, l = threadIdx.x % 64;
    __syncthreads();
    if (l == 0)
#pragma unroll
      for (int j = 0; j < N; ++j) red[j * (TPB / 64) + w] = v[j];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < N; ++j) {
      T t = red[j * (TPB / 64)];
#pragma unroll
      for (int i = 1; i < TPB / 64; ++i) t += red[j * (TPB / 64) + i];
      v[j] = t;
    }
  }
}

template <int TPB, typename T>
__device__ inline T block_max(T v, T *red) {
  v = wave_max(v);
  if constexpr (TPB == 64) {
    return v;
  } else {
    const int w = threadIdx.x / 64, l = threadIdx.x % 64;
    __syncthreads();
    if (l == 0) red[w] = v;
    __syncthreads();
    T t = red[0];
#pragma unroll
    for (int i = 1; i < TPB / 64; ++i) t = fmax(t, red[i]);
    return t;
  }
}

// A value equal in all lanes of the wave, held as such: branches on it and the
// addresses formed from it are scalar.
__device__ inline int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ inline bool uniform(bool v) { return __builtin_amdgcn_readfirstlane((int)v) != 0; }
__device__ inline int64_t uniform(int64_t v) {
  const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(uint64_t)v);
  const unsigned hi = (unsigned)__builtin_amdgcn_readfirstlane((int)((uint64_t)v >> 32));
  return (int64_t)(((uint64_t)hi << 32) | lo);
}

// Lane k's value (k uniform), in scalar registers.
__device__ inline float wave_value(float v, int k) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), k));
}
__device__ inline double wave_value(double v, int k) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), k),
                          __builtin_amdgcn_readlane(__double2loint(v), k));
}

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }
inline size_t align_up(size_t x, size_t a = 256) { return (x + a - 1) / a * a; }

// Bump allocator over a caller-provided workspace.
struct Arena {
  char *base = nullptr;
  size_t cap = 0, off = 0;
  bool measure = false;  // only count bytes
  Arena() = default;
  Arena(void *b, size_t c) : base((char *)b), cap(c), off(0), measure(b == nullptr) {}
  template <typename T>
  T *take(size_t n) {
    size_t o = align_up(off);
    off = o + n * sizeof(T);
    if (measure) return nullptr;
    if (off > cap) return nullptr;
    return (T *)(base + o);
  }
  bool ok() const { return measure || off <= cap; }
};

// thread-local last error
void set_error(const char *fmt, ...);
const char *last_error();

#define SB_HIP(expr)                                                                 \
  do {                                                                               \
    hipError_t _e = (expr);                                                          \
    if (_e != hipSuccess) {                                                          \
      ::sb::set_error("%s failed: %s (%s:%d)", #expr, hipGetErrorString(_e), __FILE__, \
                      __LINE__);                                                     \
      return SB_E_DEVICE;                                                            \
    }                                                                                \
  } while (0)

#define SB_LAUNCH_CHECK() SB_HIP(hipGetLastError())

}  // namespace sb
