// Mixture row scalars shared by the contraction epilogues (two-launch and
// fused paths).
#pragma once

#include "internal.h"

namespace sb {

constexpr int kMaxK = 16;

// Mixture row: q_k from its tile partials, a_k = beta_k - q_k/2, lse =
// logsumexp_k a_k and the responsibilities r_k = exp(a_k - lse) in T (FP64
// arithmetic).  Shared by the epilogue and the active-component lists, so
// both see the same zero responsibilities.
template <typename T>
__device__ inline void mixture_resp(const Model &m, const T *qp, int ntn, double &lse,
                                    T (&r)[kMaxK]) {
  const int K = m.K;
  double a[kMaxK];
  double mx = -INFINITY;
#pragma unroll
  for (int k = 0; k < kMaxK; ++k) {
    if (k < K) {
      double q = 0;
      for (int t = 0; t < ntn; ++t) q += (double)qp[k * ntn + t];
      a[k] = m.beta[k] - 0.5 * q;
      mx = fmax(mx, a[k]);
    }
  }
  if (K == 1) {
    lse = a[0];
  } else {
    double ssum = 0;
#pragma unroll
    for (int k = 0; k < kMaxK; ++k)
      if (k < K) ssum += exp(a[k] - mx);
    lse = mx + log(ssum);
  }
#pragma unroll
  for (int k = 0; k < kMaxK; ++k) r[k] = (k < K) ? (K == 1 ? (T)1 : (T)exp(a[k] - lse)) : (T)0;
}

// Component k of one wave's row in lane k: the tile partials of the K
// components are read side by side, each exp is formed once, and every lane
// adds them in component order from zero, so lse and r are the bits of
// mixture_resp.  lane_resp: lane k's r_k (zero past K).  With one component
// per lane the row waits for ntn loads and two exps instead of K ntn and 2 K.
template <typename T>
__device__ inline void mixture_resp_wave(int K, const double *beta, const T *qp, int ntn, int lane,
                                         double &lse, T &lane_resp) {
  const bool act = lane < K;
  double a = -INFINITY;
  if (act) {
    double q = 0;
#pragma unroll 4
    for (int t = 0; t < ntn; ++t) q += (double)qp[lane * ntn + t];
    a = beta[lane] - 0.5 * q;
  }
  if (K == 1) {
    lse = wave_value(a, 0);
    lane_resp = act ? (T)1 : (T)0;
    return;
  }
  const double mx = wave_max(a);
  const double e = act ? exp(a - mx) : 0.0;
  double ssum = 0;
  for (int k = 0; k < K; ++k) ssum += wave_value(e, k);
  lse = mx + log(ssum);
  lane_resp = act ? (T)exp(a - lse) : (T)0;
}

// One row per KP lanes (KP a power of two, at least K), component k in lane k
// of the row's group: the l of many rows at once, same arithmetic and order.
template <int KP, typename T>
__device__ inline double mixture_lse_group(int K, const double *beta, const T *qp, int ntn) {
  const int lane = threadIdx.x & 63, k = lane & (KP - 1), base = lane & ~(KP - 1);
  double a = -INFINITY;
  if (k < K) {
    double q = 0;
#pragma unroll 4
    for (int t = 0; t < ntn; ++t) q += (double)qp[k * ntn + t];
    a = beta[k] - 0.5 * q;
  }
  if (K == 1) return KP == 1 ? a : __shfl(a, base, 64);
  double mx = a;
#pragma unroll
  for (int o = 1; o < KP; o <<= 1) mx = fmax(mx, __shfl_xor(mx, o, 64));
  const double e = k < K ? exp(a - mx) : 0.0;
  double ssum = 0;
#pragma unroll
  for (int c = 0; c < KP; ++c) {
    const double v = __shfl(e, base + c, 64);
    if (c < K) ssum += v;
  }
  return mx + log(ssum);
}

}  // namespace sb
