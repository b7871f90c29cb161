// Batched L-BFGS on f = -l, one workgroup per start (appendix "L-BFGS
// Optimization"; batched over samples as the paper describes).
//
// Each start is a small state machine advanced once per batch step:
//   INIT      the start point has been evaluated: choose the first direction.
//   TRIAL     the trial x + alpha p has been evaluated: Armijo test
//             f(x_t) <= f(x) + 1e-4 alpha g^T p.  Accept -> store (s, y) if
//             s^T y > 1e-10 |s| |y|, compute the next direction by the
//             two-loop recursion; reject -> halve alpha (at most 40 times;
//             then clear the history and retry steepest descent once, else
//             the start is stalled).
// Starts stop when ||grad l||_inf <= tol or after max_iter accepted steps.
// The first direction, and any direction after a history reset or a
// non-descent two-loop result, is -g / max(1, ||g||_inf).
//
// Points and gradients are double-buffered per start (slots 0/1, `cur` names
// the accepted point), so accepting a trial swaps a slot index instead of
// copying.  The history S, Y [B][m][d] is a ring in memory; the kernel loads
// it into registers by age (newest first) and runs both loops of the recursion
// with workgroup reductions for the dot products.
#include <algorithm>
#include <cstdlib>

#include "fused_tile.h"
#include "internal.h"

namespace sb {

enum { PH_INIT = 0, PH_TRIAL = 1 };
enum { ST_ACTIVE = 0, ST_CONVERGED = 1, ST_STALLED = 2, ST_MAXITER = 3, ST_DEAD = 4 };

template <typename T>
struct LbArgs {
  int64_t B;
  int d, m, max_iter;
  T tol;
  T *X, *G, *Pd, *S, *Yh, *rho, *yy, *alpha, *gtp;
  double *F;  // l at both slots, FP64 for every operand type
  int32_t *cur, *head, *cnt, *iters, *ls, *status, *phase, *rowid, *active;
  // per-start vector offset and length (nullable: s * d and d), and the
  // element offset of each start's trial row (nullable)
  const int64_t *voff;
  const int32_t *vdim;
  int64_t *rowoff;
  int64_t Ltot;
  // batches: problem of each start, per-problem tolerance and iteration cap
  // (nullable: tol / max_iter), and the first start of this launch
  const int32_t *sprob;
  const double *ptol;
  const int32_t *pmaxit;
  int64_t s_base, s_count;  // starts [s_base, s_base + s_count) of this launch
  int32_t *count_reset;     // compaction count, zeroed by this launch (nullable)
  float *moved;             // FP32: |trial - its slot's old content|^2 (nullable)
};

// A thread's chunk [i0, i0 + EPT) of a length-d vector (i0 = tid * EPT), at
// whatever element the vector starts: a whole chunk is one access of 16-byte
// pieces (global memory takes them at any alignment), the chunk that crosses
// the end is taken one value at a time, and chunks past it are zero.  What the
// loads cost is their waits, so nothing in them may ask for one: zeros come first (in
// the branch that takes them they would wait for the load of the other lanes), and
// the byte offset is formed once (formed at each load it lands in the load's own
// destination).  FP64, m = 8, 4096 starts of d = 203: 46.8 -> 37.9 us, d = 401
// 97 -> 66; FP32 d = 1000 94 -> 66.
// NT: the streaming form, for the history ring and the direction, which are
// read and written once per step and not again before the whole batch has moved
// several times the size of the last-level cache: non-temporal accesses keep
// them from displacing the points and gradients the contraction reads next.
template <typename T, int N>
struct VecU {
  typedef T v __attribute__((ext_vector_type(N), aligned(sizeof(T))));
};
template <typename T, int N, bool NT>
__device__ inline void piece_load(const T *p, T *v) {
  if constexpr (N == 1) {
    v[0] = NT ? __builtin_nontemporal_load(p) : *p;
  } else {
    typedef typename VecU<T, N>::v vt;
    const vt w = NT ? __builtin_nontemporal_load((const vt *)p) : *(const vt *)p;
#pragma unroll
    for (int e = 0; e < N; ++e) v[e] = w[e];
  }
}
template <typename T, int N, bool NT>
__device__ inline void piece_store(T *p, const T *v) {
  if constexpr (N == 1) {
    if constexpr (NT)
      __builtin_nontemporal_store(v[0], p);
    else
      *p = v[0];
  } else {
    typedef typename VecU<T, N>::v vt;
    vt w;
#pragma unroll
    for (int e = 0; e < N; ++e) w[e] = v[e];
    if constexpr (NT)
      __builtin_nontemporal_store(w, (vt *)p);
    else
      *(vt *)p = w;
  }
}
// Where a thread's chunk begins: its first element, and the byte offset in a vector
// of T, which the compiler is kept from forming anew at each load (not with eight
// values a thread, whose registers are the shorter: 16384 starts of d = 1024 with
// the history in BF16 lost 7% by it).
struct ChunkAt {
  int i0;
  uint32_t off;
  template <int EPT, typename T>
  __device__ const T *at(const T *p) const {
    return EPT > 4 ? p + i0 : (const T *)((const char *)p + off);
  }
};
template <typename T, int EPT>
__device__ inline ChunkAt chunk_at(int tid) {
  ChunkAt a{tid * EPT, (uint32_t)(tid * EPT) * (uint32_t)sizeof(T)};
  if constexpr (EPT <= 4) asm volatile("" : "+v"(a.off));
  return a;
}
template <typename T, int EPT, bool NT>
__device__ inline void chunk_load(const T *p, ChunkAt at, int d, T (&v)[EPT]) {
  const T *q = at.template at<EPT>(p);
#pragma unroll
  for (int e = 0; e < EPT; ++e) v[e] = (T)0;
  if (at.i0 + EPT <= d) piece_load<T, EPT, NT>(q, v);
  if (d % EPT != 0) {  // (uniform)
    const bool part = at.i0 + EPT > d;
#pragma unroll
    for (int e = 0; e < EPT; ++e)
      if (part && at.i0 + e < d) v[e] = q[e];
  }
}
template <typename T, int EPT, bool NT>
__device__ inline void chunk_store(T *p, ChunkAt at, int d, const T (&v)[EPT]) {
  T *q = (T *)at.template at<EPT>(p);
  if (at.i0 + EPT <= d) piece_store<T, EPT, NT>(q, v);
  if (d % EPT != 0) {
    const bool part = at.i0 + EPT > d;
#pragma unroll
    for (int e = 0; e < EPT; ++e)
      if (part && at.i0 + e < d) q[e] = v[e];
  }
}
template <typename T, int EPT>
__device__ inline void vload(const T *p, ChunkAt at, int d, T (&v)[EPT]) {
  chunk_load<T, EPT, false>(p, at, d, v);
}
template <typename T, int EPT>
__device__ inline void vstore(T *p, ChunkAt at, int d, const T (&v)[EPT]) {
  chunk_store<T, EPT, false>(p, at, d, v);
}
template <typename T, int EPT>
__device__ inline void vload_nt(const T *p, ChunkAt at, int d, T (&v)[EPT]) {
  chunk_load<T, EPT, true>(p, at, d, v);
}
template <typename T, int EPT>
__device__ inline void vstore_nt(T *p, ChunkAt at, int d, const T (&v)[EPT]) {
  chunk_store<T, EPT, true>(p, at, d, v);
}

// The history ring in BF16 (FP32 starts): a thread's EPT values as EPT
// 16-bit words, widened on load (exact) and rounded to nearest on store; the
// pair is rounded before any use, so the stored values are the ones used.
__device__ inline float bf16_round(float v) {
  const __bf16 h = (__bf16)v;
  return (float)h;
}
template <int EPT>
__device__ inline void hload_nt(const uint16_t *p, int i0, int d, float (&v)[EPT]) {
  // (chunks that cross the end, and odd chunk sizes: four values at a time)
#pragma unroll
  for (int q = 0; q < EPT; q += (EPT % 4 ? 1 : 4)) {
    if (EPT % 4 == 0 && i0 + q + 4 <= d) {
      typedef uint32_t u2v __attribute__((ext_vector_type(2), aligned(2)));
      const u2v w = __builtin_nontemporal_load((const u2v *)(p + i0 + q));
      v[q] = __builtin_bit_cast(float, w[0] << 16);
      v[q + 1] = __builtin_bit_cast(float, w[0] & 0xffff0000u);
      v[q + 2] = __builtin_bit_cast(float, w[1] << 16);
      v[q + 3] = __builtin_bit_cast(float, w[1] & 0xffff0000u);
    } else {
#pragma unroll
      for (int e = q; e < q + (EPT % 4 ? 1 : 4); ++e)
        v[e] = (i0 + e < d) ? __builtin_bit_cast(float, (uint32_t)p[i0 + e] << 16) : 0.f;
    }
  }
}
template <int EPT>
__device__ inline void hstore_nt(uint16_t *p, int i0, int d, const float (&v)[EPT]) {
  // (v already holds BF16 values: the top 16 bits are exact)
  auto pk = [&](int e) {
    return (__builtin_bit_cast(uint32_t, v[e]) >> 16) |
           (__builtin_bit_cast(uint32_t, v[e + 1]) & 0xffff0000u);
  };
  if constexpr (EPT % 8 == 0) {
    if (i0 + EPT <= d) {
      typedef uint32_t u4v __attribute__((ext_vector_type(4), aligned(2)));
#pragma unroll
      for (int q = 0; q < EPT; q += 8) {
        u4v w;
#pragma unroll
        for (int e = 0; e < 4; ++e) w[e] = pk(q + 2 * e);
        __builtin_nontemporal_store(w, (u4v *)(p + i0 + q));
      }
      return;
    }
  }
#pragma unroll
  for (int q = 0; q < EPT; q += (EPT % 4 ? 1 : 4)) {
    if constexpr (EPT % 4 == 0) {
      if (i0 + q + 4 <= d) {
        typedef uint32_t u2v __attribute__((ext_vector_type(2), aligned(2)));
        u2v w;
        w[0] = pk(q);
        w[1] = pk(q + 2);
        __builtin_nontemporal_store(w, (u2v *)(p + i0 + q));
        continue;
      }
    }
#pragma unroll
    for (int e = q; e < q + (EPT % 4 ? 1 : 4); ++e)
      if (i0 + e < d) p[i0 + e] = (uint16_t)(__builtin_bit_cast(uint32_t, v[e]) >> 16);
  }
}
// The raw words of a thread's EPT BF16 values (EPT even, whole chunk), kept
// packed in registers: no conversion between the loads, so the loads of a whole
// history issue back to back.
template <int EPT>
__device__ inline void hload_raw_nt(const uint16_t *p, int i0, uint32_t (&w)[EPT / 2]) {
  static_assert(EPT % 2 == 0, "whole 32-bit words");
  constexpr int N = EPT % 8 == 0 ? 4 : (EPT % 4 == 0 ? 2 : 1);
  typedef uint32_t uv __attribute__((ext_vector_type(N), aligned(2)));
#pragma unroll
  for (int q = 0; q < EPT / 2; q += N) {
    const uv t = __builtin_nontemporal_load((const uv *)(p + i0 + 2 * q));
#pragma unroll
    for (int e = 0; e < N; ++e) w[q + e] = t[e];
  }
}
// Ring access for history type HB (BF16 when true, else T).
template <typename T, int EPT, bool HB>
__device__ inline void ring_load(const T *base, size_t off, ChunkAt at, int d, T (&v)[EPT]) {
  if constexpr (HB)
    hload_nt<EPT>((const uint16_t *)base + off, at.i0, d, v);
  else
    vload_nt<T, EPT>(base + off, at, d, v);
}
template <typename T, int EPT, bool HB>
__device__ inline void ring_store(T *base, size_t off, ChunkAt at, int d, const T (&v)[EPT]) {
  if constexpr (HB)
    hstore_nt<EPT>((uint16_t *)base + off, at.i0, d, v);
  else
    vstore_nt<T, EPT>(base + off, at, d, v);
}

// A thread's slices of the kMaxHist register-resident history vectors:
// EPT values of type T each, or (PK: FP32 starts with the history in BF16,
// EPT even) the same values packed two per 32-bit word and widened on each
// read, which halves the registers the history holds.  Values given to set
// must be BF16-exact in the packed form (the low 16 bits are dropped).
template <typename T, int EPT, bool PK>
struct HistReg {
  T v[kMaxHist][EPT];
  __device__ T get(int j, int e) const { return v[j][e]; }
  __device__ void set(int j, const T (&x)[EPT]) {
#pragma unroll
    for (int e = 0; e < EPT; ++e) v[j][e] = x[e];
  }
  __device__ void move(int j, int k) {
#pragma unroll
    for (int e = 0; e < EPT; ++e) v[j][e] = v[k][e];
  }
};
template <int EPT>
struct HistReg<float, EPT, true> {
  static_assert(EPT % 2 == 0, "two BF16 values per word");
  uint32_t w[kMaxHist][EPT / 2];
  __device__ float get(int j, int e) const {
    const uint32_t x = w[j][e >> 1];
    return __builtin_bit_cast(float, (e & 1) ? (x & 0xffff0000u) : (x << 16));
  }
  __device__ void set(int j, const float (&x)[EPT]) {
#pragma unroll
    for (int q = 0; q < EPT / 2; ++q)
      w[j][q] = (__builtin_bit_cast(uint32_t, x[2 * q]) >> 16) |
                (__builtin_bit_cast(uint32_t, x[2 * q + 1]) & 0xffff0000u);
  }
  __device__ void move(int j, int k) {
#pragma unroll
    for (int q = 0; q < EPT / 2; ++q) w[j][q] = w[k][q];
  }
};

// Workgroup reductions over a two-slot LDS ring, one barrier each (the
// summation order of block_sum: butterfly within each wave, then the wave
// totals in order, so results are the same).  Reduction k writes slot
// k & 1; a thread reaches the write of reduction k + 2 only after every
// thread has passed the barrier of reduction k + 1, that is, after every
// read of reduction k.  All threads make the same sequence of calls.
template <int TPB, typename T>
struct BlockRed {
  static constexpr int NW = TPB / 64, NMAX = 4;
  T *buf;  // LDS, 2 * NMAX * NW elements
  int slot;
  template <int N, bool MAX>
  __device__ __forceinline__ void reduce(T (&v)[N]) {
    static_assert(N <= NMAX, "values per reduction");
#pragma unroll
    for (int j = 0; j < N; ++j) v[j] = MAX ? wave_max(v[j]) : wave_sum(v[j]);
    if constexpr (NW > 1) {
      T *r = buf + slot * (NMAX * NW);
      slot ^= 1;
      const int w = threadIdx.x / 64, l = threadIdx.x % 64;
      if (l == 0)
#pragma unroll
        for (int j = 0; j < N; ++j) r[j * NW + w] = v[j];
      __syncthreads();
#pragma unroll
      for (int j = 0; j < N; ++j) {
        T t = r[j * NW];
#pragma unroll
        for (int i = 1; i < NW; ++i) t = MAX ? fmax(t, r[j * NW + i]) : t + r[j * NW + i];
        v[j] = t;
      }
    }
  }
  __device__ __forceinline__ T sum(T x) {
    T v[1] = {x};
    reduce<1, false>(v);
    return v[0];
  }
};

// Two-loop recursion on register-resident history.  Sets 1 to n hold pairs
// from newer to older, set 0 one more: the newest of all, or (old0) the
// oldest, or (cnt == n) nothing; rho of set j is in lane j.  q <- g; backward:
// alpha_j = rho_j s_j^T q, q -= alpha_j y_j; r = gamma q, gamma = s^T y / y^T y
// of the newest pair; forward: beta = rho_j y_j^T r, r += (alpha_j - beta) s_j;
// returns p = -r.
template <typename T, int TPB, int EPT, class H>
__device__ inline void two_loop(const H &Sr, const H &Yr, T rh, T gamma, int cnt, int n, bool old0,
                                const T (&g)[EPT], T (&p)[EPT], BlockRed<TPB, T> &red) {
  T q[EPT], al[kMaxHist];
#pragma unroll
  for (int e = 0; e < EPT; ++e) q[e] = g[e];
  auto back = [&](int j) {
    T dd = 0;
#pragma unroll
    for (int e = 0; e < EPT; ++e) dd += Sr.get(j, e) * q[e];
    dd = red.sum(dd);
    al[j] = wave_value(rh, j) * dd;
#pragma unroll
    for (int e = 0; e < EPT; ++e) q[e] -= al[j] * Yr.get(j, e);
  };
  auto fwd = [&](int j) {
    T bb = 0;
#pragma unroll
    for (int e = 0; e < EPT; ++e) bb += Yr.get(j, e) * q[e];
    bb = wave_value(rh, j) * red.sum(bb);
#pragma unroll
    for (int e = 0; e < EPT; ++e) q[e] += (al[j] - bb) * Sr.get(j, e);
  };
  al[0] = 0;
  if (cnt > n && !old0) back(0);
#pragma unroll
  for (int j = 1; j < kMaxHist; ++j)
    if (j <= n)
      back(j);
    else
      al[j] = 0;
  if (cnt > n && old0) back(0);
#pragma unroll
  for (int e = 0; e < EPT; ++e) q[e] *= gamma;
  if (cnt > n && old0) fwd(0);
#pragma unroll
  for (int j = kMaxHist - 1; j >= 1; --j)
    if (j <= n) fwd(j);
  if (cnt > n && !old0) fwd(0);
#pragma unroll
  for (int e = 0; e < EPT; ++e) p[e] = -q[e];
}

// The same recursion with the history left in memory, for memories beyond
// what registers hold (m up to kMaxMem).  Pair j (logical order, oldest
// first) sits at Sb + slot(j) * d and Yb + slot(j) * d with its rho at
// rho[slot(j)], slot(j) = (head - cnt + j) mod m.  The backward loop reads
// the pairs newest first, the forward loop oldest first, so each pair is
// read twice; the oldest pairs are the last read by the first loop and the
// first by the second, and the second read of a pair is its last use
// (non-temporal).  The next pair's chunks are loaded before the current
// pair's reduction so that the load latency overlaps it.  When `reg_new`,
// the newest pair (logical cnt - 1) is taken from sn, yn, rn instead.  The
// arithmetic and its order are those of two_loop.
template <typename T, int TPB, int EPT, bool LATE = false>
__device__ __forceinline__ void two_loop_stream(const T *Sb, const T *Yb, const T *rho, int d, int m,
                                       int head, int cnt, bool reg_new,
                                       const T (&sn)[EPT], const T (&yn)[EPT], T rn, T gamma,
                                       const T (&g)[EPT], T (&p)[EPT], BlockRed<TPB, T> &red) {
  const ChunkAt at = chunk_at<T, EPT>(threadIdx.x);
  T q[EPT], al[kMaxMem];
#pragma unroll
  for (int e = 0; e < EPT; ++e) q[e] = g[e];
  const int slot0 = head >= cnt ? head - cnt : head - cnt + m;
  auto slot = [&](int j) { return slot0 + j < m ? slot0 + j : slot0 + j - m; };
  // Two buffers by turns: a copy from one to the other would wait for the pair
  // under way ahead of the current one's reduction (FP64, m = 32, 1024 starts of
  // d = 199: 74 us against 56).  FP64 copies all the same where the registers of two
  // buffers cost a wave per SIMD that tells more: m = 12, 4096 starts of d = 128 44 us
  // against 36, d = 402 129 against 112.  (LATE: always.)
  constexpr bool TURNS = !LATE && (sizeof(T) == 4 || (EPT > 2 && TPB == 64));
  // LATE (rows of EPT values at least): the chunk that crosses the rows' end is loaded
  // whole from their last EPT values and shifted to its place when it is copied.  One mask
  // for the loads of all lanes, and nothing at the loads that waits for them.
  static_assert(EPT <= 4 || !LATE, "shifts by up to 3");
  const int sh = d % EPT ? EPT - d % EPT : 0;
  const bool cross = at.i0 < d && at.i0 + EPT > d;
  uint32_t loff = at.off - (cross ? (uint32_t)sh * (uint32_t)sizeof(T) : 0u);
  if constexpr (LATE) asm volatile("" : "+v"(loff));
  auto row = [&](const T *r, T (&v)[EPT], bool last) {
    if constexpr (LATE) {
      const T *q0 = (const T *)((const char *)r + loff);
#pragma unroll
      for (int e = 0; e < EPT; ++e) v[e] = (T)0;
      if (at.i0 < d) {
        if (last) piece_load<T, EPT, true>(q0, v);
        else piece_load<T, EPT, false>(q0, v);
      }
    } else if (last) {
      vload_nt<T, EPT>(r, at, d, v);
    } else {
      vload<T, EPT>(r, at, d, v);
    }
  };
  // (reg: the pair from the registers, in place already)
  auto settle = [&](const T (&v)[EPT], T (&o)[EPT], bool reg) {
    // (uniform; the branch also keeps the shift from moving up to the loads, whose wait
    // it would bring: up to 2.7 times the step's time)
    if (!LATE || sh == 0 || reg) {
#pragma unroll
      for (int e = 0; e < EPT; ++e) o[e] = v[e];
    } else {
      const bool c1 = cross && (sh & 1), c2 = cross && (sh & 2);
      T w[EPT + 2];
      w[EPT] = w[EPT + 1] = (T)0;
#pragma unroll
      for (int e = 0; e < EPT; ++e) w[e] = c1 ? (e + 1 < EPT ? v[e + 1] : (T)0) : v[e];
#pragma unroll
      for (int e = 0; e < EPT; ++e) o[e] = c2 ? w[e + 2] : w[e];
    }
  };
  auto fetch = [&](int j, T (&sv)[EPT], T (&yv)[EPT], T &rv, bool last) {
    if (reg_new && j == cnt - 1) {
#pragma unroll
      for (int e = 0; e < EPT; ++e) {
        sv[e] = sn[e];
        yv[e] = yn[e];
      }
      rv = rn;
      return;
    }
    const int ph = slot(j);
    row(Sb + (size_t)ph * d, sv, last);
    row(Yb + (size_t)ph * d, yv, last);
    rv = rho[ph];
  };
  T sb[2][EPT], yb[2][EPT], rb[2] = {0, 0};
  if (cnt > 0) {
    if (TURNS && cnt % 2 == 0)
      fetch(cnt - 1, sb[1], yb[1], rb[1], false);
    else
      fetch(cnt - 1, sb[0], yb[0], rb[0], false);
    if constexpr (LATE) {
      settle(sb[0], sb[0], reg_new);
      settle(yb[0], yb[0], reg_new);
    }
  }
#pragma unroll
  for (int j = kMaxMem - 1; j >= 0; --j) {
    if (j < cnt) {
      const int c = TURNS ? j % 2 : 0, n = 1 - c;
      T ns[EPT], ny[EPT], nr = 0;
      if (j > 0) fetch(j - 1, TURNS ? sb[n] : ns, TURNS ? yb[n] : ny, TURNS ? rb[n] : nr, false);
      T dd = 0;
#pragma unroll
      for (int e = 0; e < EPT; ++e) dd += sb[c][e] * q[e];
      dd = red.sum(dd);
      al[j] = rb[c] * dd;
#pragma unroll
      for (int e = 0; e < EPT; ++e) q[e] -= al[j] * yb[c][e];
      if (!TURNS && j > 0) {
        settle(ns, sb[0], false);
        settle(ny, yb[0], false);
        rb[0] = nr;
      }
    } else {
      al[j] = 0;
    }
  }
#pragma unroll
  for (int e = 0; e < EPT; ++e) q[e] *= gamma;
  if (cnt > 0) fetch(0, sb[0], yb[0], rb[0], true);
  if constexpr (LATE) {
    if (cnt > 0) {
      settle(sb[0], sb[0], reg_new && cnt == 1);
      settle(yb[0], yb[0], reg_new && cnt == 1);
    }
  }
#pragma unroll
  for (int j = 0; j < kMaxMem; ++j) {
    if (j < cnt) {
      const int c = TURNS ? j % 2 : 0, n = 1 - c;
      T ns[EPT], ny[EPT], nr = 0;
      if (j + 1 < cnt)
        fetch(j + 1, TURNS ? sb[n] : ns, TURNS ? yb[n] : ny, TURNS ? rb[n] : nr, true);
      T bb = 0;
#pragma unroll
      for (int e = 0; e < EPT; ++e) bb += yb[c][e] * q[e];
      bb = rb[c] * red.sum(bb);
#pragma unroll
      for (int e = 0; e < EPT; ++e) q[e] += (al[j] - bb) * sb[c][e];
      if (!TURNS && j + 1 < cnt) {
        settle(ns, sb[0], reg_new && j + 2 == cnt);
        settle(ny, yb[0], reg_new && j + 2 == cnt);
        rb[0] = nr;
      }
    }
  }
#pragma unroll
  for (int e = 0; e < EPT; ++e) p[e] = -q[e];
}

// |x - o|^2 over a start's threads.
template <typename T, int TPB, int EPT>
__device__ __forceinline__ T moved_sq(const T (&x)[EPT], const T (&o)[EPT],
                                      BlockRed<TPB, T> &red) {
  T dd = 0;
#pragma unroll
  for (int e = 0; e < EPT; ++e) {
    const T t = x[e] - o[e];
    dd += t * t;
  }
  return red.sum(dd);
}

// One step of start s by its TPB threads, tid the thread's index among them
// (every branch is uniform in s).  Returns the row of the trial point to be
// evaluated, or -1 when the start has stopped.  HREG: the history is held in
// registers (m <= kMaxHist); otherwise it stays in memory and two_loop_stream
// reads it (m <= kMaxMem).  HB (FP32, HREG): the ring holds BF16 pairs (s and y
// rounded to BF16 when formed).  MV (FP32): the distance that the trial moved its
// slot is written too; it holds the old point to the end, so only the launches
// that a screen follows have it.
template <typename T, int TPB, int EPT, bool HREG, bool HB, bool MV, bool LATE = false>
__device__ __forceinline__ int32_t lbfgs_step_one(const LbArgs<T> &a, const int64_t s,
                                                  const int tid, BlockRed<TPB, T> &red) {
  static_assert(!HB || (HREG && sizeof(T) == 4), "BF16 history: FP32, register-resident");
  const int64_t B = a.B;
  // every per-start scalar is read before the first decision, so the reads
  // share one memory round trip (all are in bounds for any start); what steers
  // the step is then the same in every lane, for the compiler too
  const int status_v = a.status[s], cur_v = a.cur[s], phase_v = a.phase[s], cnt_v = a.cnt[s],
            head_v = a.head[s], it_v = a.iters[s];
  const double f0 = a.F[s], f1 = a.F[(size_t)B + s];
  const T alpha_s = a.alpha[s], gtp_s = a.gtp[s];
  const int ls_v = a.ls[s];
  const int dv_v = a.vdim ? a.vdim[s] : a.d;
  const int64_t vo_v = a.voff ? a.voff[s] : (int64_t)s * a.d;
  const int sp_v = a.sprob ? a.sprob[s] : 0;
  const int status = uniform(status_v), phase = uniform(phase_v), ls_s = uniform(ls_v);
  int cur = uniform(cur_v), cnt = uniform(cnt_v), head = uniform(head_v), it = uniform(it_v);
  const int dv = uniform(dv_v);
  const int64_t vov = uniform(vo_v);
  if (status != ST_ACTIVE) {
    if (tid == 0) a.active[s] = 0;
    return -1;
  }
  const int m = a.m;
  const int d = dv;
  const int64_t vo = vov;
  const int64_t Lt = a.Ltot;
  const ChunkAt at = chunk_at<T, EPT>(tid);  // this thread's chunk of every vector
  T tol = a.tol;
  int max_iter = a.max_iter;
  if (a.sprob) {
    // (read with the vectors below: the first use is the convergence test)
    const int p = uniform(sp_v);
    tol = (T)a.ptol[p];
    max_iter = a.pmaxit[p];
  }
  const double lcur = cur ? f1 : f0;

  // ---- decide what this step does from the scalars alone
  enum { M_INIT, M_ACCEPT, M_BACKTRACK, M_RESET, M_STALL };
  int mode = M_INIT;
  T alpha = 1;
  int lsn = 0;
  if (phase == PH_TRIAL) {
    const double lt = cur ? f0 : f1;
    alpha = alpha_s;
    const double gtp_old = (double)gtp_s;
    const double fc = -lcur, ft = -lt;
    if (uniform(isfinite(ft) && ft <= fc + 1e-4 * (double)alpha * gtp_old)) {
      mode = M_ACCEPT;
    } else {
      lsn = ls_s + 1;
      alpha *= (T)0.5;
      if (lsn <= 40)
        mode = M_BACKTRACK;
      else
        mode = (cnt > 0) ? M_RESET : M_STALL;
    }
  }
  if (mode == M_STALL) {
    if (tid == 0) {
      a.status[s] = ST_STALLED;
      a.active[s] = 0;
    }
    return -1;
  }
  if (mode == M_BACKTRACK) {
    const int tr = 1 - cur;
    const T *xc = a.X + (size_t)cur * Lt + vo;
    T *xt = a.X + (size_t)tr * Lt + vo;
    const T *pd = a.Pd + vo;
    T c[EPT], q[EPT];
    vload<T, EPT>(xc, at, d, c);
    vload<T, EPT>(pd, at, d, q);
#pragma unroll
    for (int e = 0; e < EPT; ++e) c[e] = c[e] + alpha * q[e];
    if constexpr (MV) {
      T o[EPT];
      vload<T, EPT>(xt, at, d, o);
      const T dd = moved_sq<T, TPB, EPT>(c, o, red);
      if (tid == 0) a.moved[(size_t)tr * B + s] = dd;
    }
    vstore<T, EPT>(xt, at, d, c);
    if (tid == 0) {
      a.alpha[s] = alpha;
      a.ls[s] = lsn;
      a.active[s] = 1;
      a.rowid[s] = (int32_t)((size_t)tr * B + s);
      if (a.rowoff) a.rowoff[s] = (int64_t)tr * Lt + vo;
    }
    return (int32_t)((size_t)tr * B + s);
  }

  // ---- load the point whose direction we now compute (and, on accept, the old one)
  T x[EPT], gl[EPT], sv[EPT], yv[EPT];
  [[maybe_unused]] T xold[MV ? EPT : 1];  // (accepted: the old point, in the trial's slot)
  const int newcur = (mode == M_ACCEPT) ? 1 - cur : cur;
  {
    const T *xn = a.X + (size_t)newcur * Lt + vo;
    const T *gn = a.G + (size_t)newcur * Lt + vo;
    const T *xo = a.X + (size_t)cur * Lt + vo;
    const T *go = a.G + (size_t)cur * Lt + vo;
    vload<T, EPT>(xn, at, d, x);
    vload<T, EPT>(gn, at, d, gl);
    if (mode == M_ACCEPT) {
      T xov[EPT], gov[EPT];
      vload<T, EPT>(xo, at, d, xov);
      vload<T, EPT>(go, at, d, gov);
#pragma unroll
      for (int e = 0; e < EPT; ++e) {
        sv[e] = x[e] - xov[e];
        yv[e] = gov[e] - gl[e];  // grad f(x_t) - grad f(x), grad f = -grad l
        if constexpr (MV) xold[e] = xov[e];
        if constexpr (HB) {
          sv[e] = bf16_round(sv[e]);
          yv[e] = bf16_round(yv[e]);
        }
      }
    }
  }
  if (mode == M_RESET) {
    cnt = 0;
    head = 0;
  }
  // History by age (loads issued before the reductions below): pair j, j = 0
  // the newest, sits in register set j + 1, where it belongs once this step's
  // pair is in set 0; the pair that this evicts (the ring full) is not read.
  // rho of set j is in lane j, for the recursion to take, and of y^T y only the
  // newest pair's is needed: as sixteen values equal in every lane the two held
  // 32 registers in FP64, and a set chosen at run time for the new pair, with
  // the sets moved down for it, 40 to 80 more.  Should the curvature test refuse the pair, set 0
  // takes the oldest pair where the ring is full, and is left out otherwise.
  constexpr bool PK = HB && EPT % 2 == 0;
  HistReg<T, EPT, PK> Sr, Yr;
  T rh = 0, yynew = 0;
  const int lane = tid & 63;
  int nset = 0;
  bool old0 = false;
  const size_t hist0 = (size_t)m * vo;
  const T *rho_s = a.rho + (size_t)s * m, *yy_s = a.yy + (size_t)s * m;
  auto slot = [&](int age) { return head - 1 - age >= 0 ? head - 1 - age : head - 1 - age + m; };
  if constexpr (HREG) {
    // packed BF16 history in whole chunks: the raw words go straight
    // to registers, every load issued before the first use
    const bool raw = PK && at.i0 + EPT <= d;
    if (mode == M_ACCEPT) nset = cnt < m ? cnt : m - 1;
#pragma unroll
    for (int j = 1; j < kMaxHist; ++j) {
      if (j <= nset) {
        const size_t off = hist0 + (uint32_t)(slot(j - 1) * d);  // (m, d <= 32, 4096)
        if constexpr (PK) {
          if (raw) {
            hload_raw_nt<EPT>((const uint16_t *)a.S + off, at.i0, Sr.w[j]);
            hload_raw_nt<EPT>((const uint16_t *)a.Yh + off, at.i0, Yr.w[j]);
          } else {
            T t[EPT];
            ring_load<T, EPT, HB>(a.S, off, at, d, t);
            Sr.set(j, t);
            ring_load<T, EPT, HB>(a.Yh, off, at, d, t);
            Yr.set(j, t);
          }
        } else {
          ring_load<T, EPT, HB>(a.S, off, at, d, Sr.v[j]);
          ring_load<T, EPT, HB>(a.Yh, off, at, d, Yr.v[j]);
        }
      }
    }
    if (mode == M_ACCEPT && cnt > 0) {
      if (lane >= 1 && lane <= nset) rh = rho_s[slot(lane - 1)];
      yynew = yy_s[slot(0)];
    }
  }
  // streamed history: the pair pushed in this step stays in registers
  bool reg_new = false;
  T r_new = 0, yy_new = 1;
  if (mode == M_ACCEPT) {
    T v3[3] = {0, 0, 0};
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
      v3[0] += sv[e] * yv[e];
      v3[1] += sv[e] * sv[e];
      v3[2] += yv[e] * yv[e];
    }
    red.template reduce<3, false>(v3);
    const T sy = v3[0], ss = v3[1], yy = v3[2];
    cur = newcur;
    ++it;
    if (uniform(sy > (T)1e-10 * sqrt(ss) * sqrt(yy))) {
      const T rnew = (T)1 / sy;
      // store the pair in the ring and append it to the logical history
      ring_store<T, EPT, HB>(a.S, (size_t)m * vo + (size_t)head * d, at, d, sv);
      ring_store<T, EPT, HB>(a.Yh, (size_t)m * vo + (size_t)head * d, at, d, yv);
      if (tid == 0) {
        a.rho[(size_t)s * m + head] = rnew;
        a.yy[(size_t)s * m + head] = yy;
      }
      const bool full = (cnt == m);
      if constexpr (HREG) {
        Sr.set(0, sv);
        Yr.set(0, yv);
        if (lane == 0) rh = rnew;
        yynew = yy;
      } else {
        reg_new = true;
        r_new = rnew;
        yy_new = yy;
      }
      head = head + 1 < m ? head + 1 : 0;
      cnt = full ? m : cnt + 1;
    } else if (cnt == m) {
      if constexpr (HREG) {
        // (its slot is the one that the refused pair would have taken)
        old0 = true;
        T t[EPT];
        ring_load<T, EPT, HB>(a.S, hist0 + (size_t)head * d, at, d, t);
        Sr.set(0, t);
        ring_load<T, EPT, HB>(a.Yh, hist0 + (size_t)head * d, at, d, t);
        Yr.set(0, t);
        if (lane == 0) rh = rho_s[head];
      }
    }
  }

  // ---- convergence tests at the current point
  // ||grad l||_inf; a non-finite entry makes it NaN (no convergence on NaN)
  T gn = 0, bad = 0;
#pragma unroll
  for (int e = 0; e < EPT; ++e) {
    gn = fmax(gn, fabs(gl[e]));
    if (!isfinite(gl[e])) bad = 1;
  }
  {
    T v2[2] = {gn, bad};
    red.template reduce<2, true>(v2);
    gn = v2[0];
    if (v2[1] != (T)0) gn = (T)NAN;
  }
  int newst = ST_ACTIVE;
  if (mode == M_INIT && uniform(!(isfinite(lcur) && isfinite(gn))))
    newst = ST_DEAD;
  else if (uniform(gn <= tol))
    newst = ST_CONVERGED;
  else if (it >= uniform(max_iter))
    newst = ST_MAXITER;
  if (newst != ST_ACTIVE) {
    if (tid == 0) {
      a.status[s] = newst;
      a.active[s] = 0;
      a.cur[s] = cur;
      a.cnt[s] = cnt;
      a.head[s] = head;
      a.iters[s] = it;
    }
    return -1;
  }

  // ---- next direction
  T g[EPT], p[EPT];
#pragma unroll
  for (int e = 0; e < EPT; ++e) g[e] = -gl[e];
  T gtp = 0;
  bool sd = (cnt == 0);
  if (!sd) {
    // gamma = s^T y / y^T y of the newest pair (logical index cnt - 1)
    T rnew;
    if constexpr (HREG) {
      rnew = wave_value(rh, nset > 0 && (old0 || cnt == nset) ? 1 : 0);
    } else {
      if (reg_new) {
        rnew = r_new;
        yynew = yy_new;
      } else {
        const int ph = (head - 1 + m) % m;
        rnew = a.rho[(size_t)s * m + ph];
        yynew = a.yy[(size_t)s * m + ph];
      }
    }
    const T gamma = ((T)1 / rnew) / yynew;
    if constexpr (HREG)
      two_loop<T, TPB, EPT>(Sr, Yr, rh, gamma, cnt, nset, old0, g, p, red);
    else
      two_loop_stream<T, TPB, EPT, LATE>(a.S + (size_t)m * vo, a.Yh + (size_t)m * vo,
                                         a.rho + (size_t)s * m, d, m, head, cnt, reg_new, sv,
                                         yv, r_new, gamma, g, p, red);
    T t = 0;
#pragma unroll
    for (int e = 0; e < EPT; ++e) t += g[e] * p[e];
    gtp = red.sum(t);
    if (uniform(!(gtp < (T)0))) {
      sd = true;
      cnt = 0;
      head = 0;
    }
  }
  if (sd) {
    const T sc = (T)1 / (gn > (T)1 ? gn : (T)1);
    T t = 0;
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
      p[e] = -g[e] * sc;
      t += g[e] * p[e];
    }
    gtp = red.sum(t);
  }
  const int tr = 1 - cur;
  T *xt = a.X + (size_t)tr * Lt + vo;
  T *pd = a.Pd + vo;
  T xtv[EPT];
#pragma unroll
  for (int e = 0; e < EPT; ++e) xtv[e] = x[e] + p[e];
  if constexpr (MV) {
    if (mode != M_ACCEPT) vload<T, EPT>(xt, at, d, xold);
    const T dd = moved_sq<T, TPB, EPT>(xtv, xold, red);
    if (tid == 0) a.moved[(size_t)tr * B + s] = dd;
  }
  vstore_nt<T, EPT>(pd, at, d, p);
  vstore<T, EPT>(xt, at, d, xtv);
  if (tid == 0) {
    a.alpha[s] = (T)1;
    a.gtp[s] = gtp;
    a.ls[s] = 0;
    a.cur[s] = cur;
    a.cnt[s] = cnt;
    a.head[s] = head;
    a.iters[s] = it;
    a.phase[s] = PH_TRIAL;
    a.active[s] = 1;
    a.rowid[s] = (int32_t)((size_t)tr * B + s);
    if (a.rowoff) a.rowoff[s] = (int64_t)tr * Lt + vo;
  }
  return (int32_t)((size_t)tr * B + s);
}

// Start s_base + blockIdx.x: a workgroup each.  (Four one-wave starts per
// workgroup, for d <= 256, measured the same: handing out workgroups is not what
// a step with few active starts costs.)
// Two waves per SIMD at least, which the FP64 step of up to 4 values a thread
// has without spilling (190 registers; with the history in logical order 310,
// or 256 and spilled).  FP64, m = 8: d = 256, 8192 starts 81 -> 73 us (21
// vectors moved: 69 us at the copy rate); d = 30, 32768 starts 97 -> 59 us.
template <typename T, int TPB, int EPT, bool HREG, bool HB, bool MV>
__global__ __launch_bounds__(TPB, 2) void lbfgs_step_kernel(LbArgs<T> a) {
  __shared__ T rbuf[2 * BlockRed<TPB, T>::NMAX * (TPB / 64)];
  BlockRed<TPB, T> red{rbuf, 0};
  // the compaction that follows counts from zero; every reader of the
  // previous count ran before this launch
  if (a.count_reset && blockIdx.x == 0 && threadIdx.x == 0) *a.count_reset = 0;
  if ((int64_t)blockIdx.x < a.s_count)
    lbfgs_step_one<T, TPB, EPT, HREG, HB, MV>(a, a.s_base + blockIdx.x, threadIdx.x, red);
}

// The step of FP64 starts with a long streamed history whose rows end inside a thread's
// values (two_loop_stream's LATE).  Loaded under a second mask, such a chunk makes each copy
// there wait more than once, and two buffers by turns cost a wave per SIMD: m = 32, 1024
// starts of d = 127 49 -> 35 us, d = 203 57 -> 44, d = 331 90 -> 58, d = 402 86 -> 64, d = 511
// 103 -> 80, d = 1002 222 -> 192, d = 2047 422 -> 344; m = 16, d = 511 53 -> 45.  Up to m = 12
// the shifts cost as much (m = 10, 1025 starts of d = 257 25 -> 27).
template <int TPB, int EPT>
__global__ __launch_bounds__(TPB, TPB == 512 ? 2 : EPT == 4 ? 3 : 4)
void lbfgs_step_ragged_kernel(LbArgs<double> a) {
  __shared__ double rbuf[2 * BlockRed<TPB, double>::NMAX * (TPB / 64)];
  BlockRed<TPB, double> red{rbuf, 0};
  if (a.count_reset && blockIdx.x == 0 && threadIdx.x == 0) *a.count_reset = 0;
  if ((int64_t)blockIdx.x < a.s_count)
    lbfgs_step_one<double, TPB, EPT, false, false, false, true>(a, a.s_base + blockIdx.x,
                                                                threadIdx.x, red);
}

template <typename T, int TPB, int EPT, bool HREG, bool HB>
static void step_go(const LbArgs<T> &a, hipStream_t s) {
  if constexpr (sizeof(T) == 4) {
    if (a.moved) {
      hipLaunchKernelGGL((lbfgs_step_kernel<T, TPB, EPT, HREG, HB, true>),
                         dim3((unsigned)a.s_count), dim3(TPB), 0, s, a);
      return;
    }
  }
  hipLaunchKernelGGL((lbfgs_step_kernel<T, TPB, EPT, HREG, HB, false>), dim3((unsigned)a.s_count),
                     dim3(TPB), 0, s, a);
}

// Workgroup size and elements per thread by d; HR: history in registers.
template <typename T, bool HR>
static void step_by_d(const LbArgs<T> &a, int d, hipStream_t s) {
  if constexpr (sizeof(T) == 8 && !HR) {
    if (!a.vdim && d > 64 && d <= 2048 && d % (d <= 128 ? 2 : 4) != 0 && a.m > 12) {
      auto go = [&](auto kernel, int tpb) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)a.s_count), dim3(tpb), 0, s, a);
      };
      if (d <= 128) go(lbfgs_step_ragged_kernel<64, 2>, 64);
      else if (d <= 256) go(lbfgs_step_ragged_kernel<64, 4>, 64);
      else if (d <= 512) go(lbfgs_step_ragged_kernel<128, 4>, 128);
      else if (d <= 1024) go(lbfgs_step_ragged_kernel<256, 4>, 256);
      else go(lbfgs_step_ragged_kernel<512, 4>, 512);
      return;
    }
  }
  if (d <= 64) step_go<T, 64, 1, HR, false>(a, s);
  else if (d <= 128) step_go<T, 64, 2, HR, false>(a, s);
  else if (d <= 256) step_go<T, 64, 4, HR, false>(a, s);
  else if (d <= 512) step_go<T, 128, 4, HR, false>(a, s);
  else if (d <= 1024) step_go<T, 256, 4, HR, false>(a, s);
  else if (d <= 2048) step_go<T, 512, 4, HR, false>(a, s);
  else step_go<T, 1024, 4, HR, false>(a, s);
}
// Register-resident history for m <= kMaxHist, streamed beyond.
template <typename T>
static void step_launch(const LbArgs<T> &a, int d, hipStream_t s) {
  if (a.m <= kMaxHist) step_by_d<T, true>(a, d, s);
  else step_by_d<T, false>(a, d, s);
}
// FP32 starts with the BF16 history ring (register-resident, m <= kMaxHist).
static void step_launch_hb(const LbArgs<float> &a, int d, hipStream_t s) {
  if (d <= 64) step_go<float, 64, 1, true, true>(a, s);
  else if (d <= 128) step_go<float, 64, 2, true, true>(a, s);
  else if (d <= 256) step_go<float, 64, 4, true, true>(a, s);
  else if (d <= 512) step_go<float, 64, 8, true, true>(a, s);
  else if (d <= 1024) step_go<float, 128, 8, true, true>(a, s);
  else if (d <= 2048) step_go<float, 256, 8, true, true>(a, s);
  else step_go<float, 512, 8, true, true>(a, s);
}

// Two-loop direction only, for B independent histories given in logical
// order (used to check the recursion in isolation).
template <typename T, int TPB, int EPT, bool HREG>
__global__ __launch_bounds__(TPB) void two_loop_kernel(int d, int m, const int32_t *cntv,
                                                       const T *S, const T *Y, const T *G, T *P) {
  const int64_t b = blockIdx.x;
  const int tid = threadIdx.x;
  __shared__ T rbuf[2 * BlockRed<TPB, T>::NMAX * (TPB / 64)];
  BlockRed<TPB, T> red{rbuf, 0};
  const int cnt = min(max(cntv[b], 0), m);  // never read past this start's m slots
  if constexpr (!HREG) {
    // rho_j and gamma from one pass over the pairs, then the streamed
    // recursion (logical order is the slot order: head = cnt mod m)
    __shared__ T rho_s[kMaxMem];
    const ChunkAt at = chunk_at<T, EPT>(tid);
    T g[EPT], p[EPT], z[EPT], gamma = 1;
#pragma unroll
    for (int e = 0; e < EPT; ++e) z[e] = 0;
    vload<T, EPT>(G + (size_t)b * d, at, d, g);
    for (int j = 0; j < cnt; ++j) {
      T sv[EPT], yv[EPT];
      vload<T, EPT>(S + ((size_t)b * m + j) * d, at, d, sv);
      vload<T, EPT>(Y + ((size_t)b * m + j) * d, at, d, yv);
      T v2[2] = {0, 0};
#pragma unroll
      for (int e = 0; e < EPT; ++e) {
        v2[0] += sv[e] * yv[e];
        v2[1] += yv[e] * yv[e];
      }
      red.template reduce<2, false>(v2);
      if (tid == 0) rho_s[j] = (T)1 / v2[0];
      if (j == cnt - 1) gamma = v2[0] / v2[1];
    }
    __syncthreads();
    two_loop_stream<T, TPB, EPT>(S + (size_t)b * m * d, Y + (size_t)b * m * d, rho_s, d, m,
                                 cnt % m, cnt, false, z, z, (T)0, gamma, g, p, red);
    vstore<T, EPT>(P + (size_t)b * d, at, d, p);
    return;
  }
  HistReg<T, EPT, false> Sr, Yr;
  T rh = 0, g[EPT], p[EPT];
  T gamma = 1;
  const ChunkAt at = chunk_at<T, EPT>(tid);
  vload<T, EPT>(G + (size_t)b * d, at, d, g);
#pragma unroll
  for (int j = 0; j < kMaxHist; ++j) {
    if (j < cnt) {
      vload<T, EPT>(S + ((size_t)b * m + (cnt - 1 - j)) * d, at, d, Sr.v[j]);
      vload<T, EPT>(Y + ((size_t)b * m + (cnt - 1 - j)) * d, at, d, Yr.v[j]);
      T v2[2] = {0, 0};
#pragma unroll
      for (int e = 0; e < EPT; ++e) {
        v2[0] += Sr.v[j][e] * Yr.v[j][e];
        v2[1] += Yr.v[j][e] * Yr.v[j][e];
      }
      red.template reduce<2, false>(v2);
      if ((tid & 63) == j) rh = (T)1 / v2[0];
      if (j == 0) gamma = v2[0] / v2[1];
    }
  }
  two_loop<T, TPB, EPT>(Sr, Yr, rh, gamma, cnt, cnt > 0 ? cnt - 1 : 0, false, g, p, red);
  vstore<T, EPT>(P + (size_t)b * d, at, d, p);
}

// ------------------------------------------------------------- dispatch

// Workgroup size and elements per thread by d; HR: history in registers.
#define SB_LB_CASES_H(KERNEL, T, HR, ...)                                                     \
  if (d <= 64) {                                                                              \
    hipLaunchKernelGGL((KERNEL<T, 64, 1, HR>), dim3((unsigned)B), dim3(64), 0, s, __VA_ARGS__);   \
  } else if (d <= 128) {                                                                      \
    hipLaunchKernelGGL((KERNEL<T, 64, 2, HR>), dim3((unsigned)B), dim3(64), 0, s, __VA_ARGS__);   \
  } else if (d <= 256) {                                                                      \
    hipLaunchKernelGGL((KERNEL<T, 64, 4, HR>), dim3((unsigned)B), dim3(64), 0, s, __VA_ARGS__);   \
  } else if (d <= 512) {                                                                      \
    hipLaunchKernelGGL((KERNEL<T, 128, 4, HR>), dim3((unsigned)B), dim3(128), 0, s, __VA_ARGS__); \
  } else if (d <= 1024) {                                                                     \
    hipLaunchKernelGGL((KERNEL<T, 256, 4, HR>), dim3((unsigned)B), dim3(256), 0, s, __VA_ARGS__); \
  } else if (d <= 2048) {                                                                     \
    hipLaunchKernelGGL((KERNEL<T, 512, 4, HR>), dim3((unsigned)B), dim3(512), 0, s, __VA_ARGS__); \
  } else {                                                                                    \
    hipLaunchKernelGGL((KERNEL<T, 1024, 4, HR>), dim3((unsigned)B), dim3(1024), 0, s,          \
                       __VA_ARGS__);                                                          \
  }
// Register-resident history for m <= kMaxHist, streamed beyond.
#define SB_LB_CASES(KERNEL, T, M, ...)              \
  if ((M) <= kMaxHist) {                            \
    SB_LB_CASES_H(KERNEL, T, true, __VA_ARGS__)     \
  } else {                                          \
    SB_LB_CASES_H(KERNEL, T, false, __VA_ARGS__)    \
  }
static int check_d(int d, int m) {
  if (d < 1 || d > 4096) {
    set_error("L-BFGS supports 1 <= d <= 4096 (got %d)", d);
    return SB_E_UNSUPPORTED;
  }
  if (m < 1 || m > kMaxMem) {
    set_error("L-BFGS memory m must be in [1, %d] (got %d)", kMaxMem, m);
    return SB_E_INVAL;
  }
  return SB_OK;
}
static int check_hist(const LbfgsBuffers &b) {
  if (b.hist_bf16 && (b.dtype != DT_F32 || b.m > kMaxHist)) {
    set_error("BF16 history needs FP32 starts and m <= %d (got m = %d)", kMaxHist, b.m);
    return SB_E_UNSUPPORTED;
  }
  return SB_OK;
}

template <typename T>
static LbArgs<T> make_args(const LbfgsBuffers &b, int max_iter, double tol) {
  LbArgs<T> a;
  a.B = b.B;
  a.d = b.d;
  a.m = b.m;
  a.max_iter = max_iter;
  a.tol = (T)tol;
  a.X = (T *)b.X;
  a.G = (T *)b.G;
  a.F = (double *)b.F;
  a.Pd = (T *)b.Pd;
  a.S = (T *)b.S;
  a.Yh = (T *)b.Yh;
  a.rho = (T *)b.rho;
  a.yy = (T *)b.yy;
  a.alpha = (T *)b.alpha;
  a.gtp = (T *)b.gtp;
  a.cur = b.cur;
  a.head = b.head;
  a.cnt = b.cnt;
  a.iters = b.iters;
  a.ls = b.ls;
  a.status = b.status;
  a.phase = b.phase;
  a.rowid = b.rowid;
  a.active = b.active;
  a.voff = b.voff;
  a.vdim = b.vdim;
  a.rowoff = b.rowoff;
  a.Ltot = b.voff ? b.Ltot : b.B * (int64_t)b.d;
  a.sprob = b.sprob;
  a.ptol = b.ptol;
  a.pmaxit = b.pmaxit;
  a.s_base = 0;
  a.s_count = b.B;
  a.count_reset = nullptr;
  a.moved = sizeof(T) == 4 ? b.moved : nullptr;
  return a;
}

// Every start of the launch has its own workgroup: the dispatcher hands freed
// slots to the next start, which balances starts of uneven cost (a fixed
// grid striding over starts measured slower: its last round runs part-empty).
int launch_lbfgs_step_range(const LbfgsBuffers &b, int64_t s_begin, int64_t count, int d_class,
                            double grad_tol, int max_iter, hipStream_t s) {
  int st = check_d(d_class, b.m);
  if (!st) st = check_hist(b);
  if (st) return st;
  if (count <= 0) return SB_OK;
  if (s_begin < 0 || s_begin + count > b.B) {
    set_error("start range [%lld, %lld) outside [0, %lld)", (long long)s_begin,
              (long long)(s_begin + count), (long long)b.B);
    return SB_E_INVAL;
  }
  auto run = [&](auto a, auto launch) {
    a.s_base = s_begin;
    a.s_count = count;
    // (the uniform batch resets its compaction count; the grouped one has its own)
    if (!b.voff) a.count_reset = b.count;
    launch(a, d_class, s);
  };
  if (b.dtype == DT_F64)
    run(make_args<double>(b, max_iter, grad_tol), step_launch<double>);
  else if (b.hist_bf16)
    run(make_args<float>(b, max_iter, grad_tol), step_launch_hb);
  else
    run(make_args<float>(b, max_iter, grad_tol), step_launch<float>);
  SB_LAUNCH_CHECK();
  return SB_OK;
}

int launch_lbfgs_step(const LbfgsBuffers &b, int max_iter, double grad_tol, hipStream_t s) {
  return launch_lbfgs_step_range(b, 0, b.B, b.d, grad_tol, max_iter, s);
}

// ---------------------------------------------------- small FP64 problems
//
// The whole iteration of 16 starts by one workgroup: a wave per start for the
// step, then the 16 trial points together on the matrix cores, until every
// start has stopped or n_steps are done.  The starts of different workgroups
// have nothing to exchange, so neither the launches of a step (step,
// compaction, evaluation) nor the readback of the active count lie between one
// step and the next; the arithmetic is theirs, in their order.  A step is
// bound by its latency: scalars, vectors, the recursion's chain of wave sums,
// the tile's loads, products and row sums.
// Bulk phase of 80 steps before and after (us): d = 4, K = 1, 64 starts 351 ->
// 238 (24 steps); d = 64, K = 4, 4096 starts 2440 -> 1310; d = 128, K = 3,
// 2048 starts 3072 -> 1925.
// prog[w]: steps workgroup w has done, or ~steps once all of its starts have
// stopped (zero before the first launch); tmax: the largest number of steps
// that any workgroup needs as far as known (one more than it has done while a
// start is active); evals: the evaluations are added.
// Starts (waves) per workgroup: 16 fill the tile; the step of two values a
// lane needs more than the 128 registers that 16 waves leave (80 of them
// spilled: 14 against 11 us a step at d = 128), so it takes 8.
template <int EPT>
constexpr int kBulkWaves = EPT == 1 ? fused::kRows : fused::kRows / 2;
struct BulkArgs {
  LbArgs<double> lb;
  Model m;
  int dp, n_steps, max_steps;
  int32_t *prog, *tmax;
  int64_t *evals;
};
struct SlotRows {  // tile row i: the row in LDS
  const int32_t *slot;
  template <int N>
  __device__ __forceinline__ void src(const int (&i)[N], int64_t (&row)[N]) const {
#pragma unroll
    for (int u = 0; u < N; ++u) row[u] = slot[i[u] < fused::kRows ? i[u] : 0];
  }
  __device__ __forceinline__ int64_t dst(int i) const { return slot[i]; }
  __device__ __forceinline__ int64_t aux(int i) const { return i; }
};
template <int EPT, int NS, bool FAST>
__global__ __launch_bounds__(64 * kBulkWaves<EPT>) void lbfgs_bulk_kernel(BulkArgs b) {
  constexpr int W = kBulkWaves<EPT>;
  extern __shared__ __attribute__((aligned(16))) double lds[];
  __shared__ int32_t slot[fused::kRows];
  __shared__ int32_t nev_s[W];
  const int t0 = uniform(b.prog[blockIdx.x]);
  if (t0 < 0) return;
  const int lane = threadIdx.x & 63, wave = uniform((int)(threadIdx.x >> 6));
  const int64_t s = (int64_t)blockIdx.x * W + wave;
  if (threadIdx.x < fused::kRows) slot[threadIdx.x] = -1;  // (rows past the waves: none)
  __syncthreads();
  BlockRed<64, double> red{nullptr, 0};  // (sums within a wave: no LDS)
  const int tend = min(t0 + b.n_steps, b.max_steps);
  int t = t0, nev = 0;
  bool done = false;
  while (t < tend) {
    // (the thread's index opaque in each iteration: what follows from it, which
    // the step and the tile form anew, else fills the registers of both)
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    int32_t row = -1;
    if (s < b.lb.B) row = lbfgs_step_one<double, 64, EPT, true, false, false>(b.lb, s, tid & 63, red);
    asm volatile("" : "+v"(tid));
    if (lane == 0) slot[wave] = row;
    nev += row >= 0;
    ++t;
    __syncthreads();  // the rows and the trial points are there
    if (!__any(slot[lane & (fused::kRows - 1)] >= 0)) {
      done = true;
      break;
    }
    fused::tile<64 * W, NS, FAST>(b.m, b.dp, b.lb.X, b.lb.d, SlotRows{slot}, b.lb.F, b.lb.G,
                                        b.lb.d, nullptr, lds, t == t0 + 1, tid);
    __syncthreads();  // l and the gradients are there, the rows read
  }
  if (lane == 0) nev_s[wave] = nev;
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long n = 0;
    for (int w = 0; w < W; ++w) n += (unsigned)nev_s[w];
    if (n) atomicAdd((unsigned long long *)b.evals, n);
    b.prog[blockIdx.x] = done ? ~t : t;
    atomicMax(b.tmax, done ? t : t + 1);
  }
}

template <int EPT, int NS>
static void bulk_go(const BulkArgs &a, bool fast, hipStream_t s) {
  const dim3 grid((unsigned)ceil_div(a.lb.B, kBulkWaves<EPT>)), block(64 * kBulkWaves<EPT>);
  const size_t lds = fused::lds_bytes(a.m.K, a.dp);
  if (fast)
    hipLaunchKernelGGL((lbfgs_bulk_kernel<EPT, NS, true>), grid, block, lds, s, a);
  else
    hipLaunchKernelGGL((lbfgs_bulk_kernel<EPT, NS, false>), grid, block, lds, s, a);
}

// Where all workgroups run at once, or nearly: there is one per CU of 256 (16
// waves at 128 registers, 8 at 170), so d <= 64 has 4096 starts in one round
// and d <= 128 2048.  Past that the launches a step that compact the starts win
// back what the last rounds, with few starts left, lose: whole calls (us, step
// launches against one launch) d = 64, K = 4 4420 : 3608 at 8192 starts, d = 16,
// K = 4 2808 : 2574 at 8192 and 3998 : 4296 at 16384; d = 128, K = 3 4156 : 3036
// at 2048, 5004 : 4992 at 4096 and 7155 : 8900 at 8192.
bool lbfgs_bulk_ok(const LbfgsBuffers &b, const Model &m) {
  const char *e = getenv("SB_ONE_LAUNCH");  // "0": the step launches (for comparison)
  if (e && e[0] == '0') return false;
  ASrc a;
  a.X = b.X;
  a.ldx = b.d;
  return b.dtype == DT_F64 && !b.hist_bf16 && !b.voff && b.m <= kMaxHist && b.d == m.d &&
         b.B <= (m.d <= 64 ? 8192 : 2048) && fused_logl_grad_ok(m, a);
}

int launch_lbfgs_bulk(const LbfgsBuffers &b, const Model &m, int max_iter, double grad_tol,
                      int n_steps, int max_steps, hipStream_t s) {
  if (!lbfgs_bulk_ok(b, m) || m.d > 128) {
    set_error("L-BFGS in one launch: unsupported model or buffers");
    return SB_E_UNSUPPORTED;
  }
  if (b.B <= 0) return SB_OK;
  BulkArgs a;
  a.lb = make_args<double>(b, max_iter, grad_tol);
  a.m = m;
  a.dp = (m.d + 31) / 32 * 32;
  a.n_steps = n_steps;
  a.max_steps = max_steps;
  a.prog = b.idx;
  a.tmax = b.count;
  a.evals = b.evals;
  const bool fast = m.d % 8 == 0 && ((uintptr_t)m.P64 & 15) == 0;
  const int nb = m.K * (a.dp / 16);  // 16-column blocks: up to 24, over the waves
  if (m.d <= 64) {
    if (nb <= 16) bulk_go<1, 1>(a, fast, s);
    else bulk_go<1, 2>(a, fast, s);
  } else {
    if (nb <= 8) bulk_go<2, 1>(a, fast, s);
    else if (nb <= 16) bulk_go<2, 2>(a, fast, s);
    else bulk_go<2, 3>(a, fast, s);
  }
  SB_LAUNCH_CHECK();
  return SB_OK;
}

int launch_two_loop(int64_t B, int d, int m, const int32_t *cnt, const void *S, const void *Y,
                    const void *G, void *P, int dtype, hipStream_t s) {
  int st = check_d(d, m);
  if (st) return st;
  if (B <= 0) return SB_OK;
  if (dtype == DT_F64) {
    SB_LB_CASES(two_loop_kernel, double, m, d, m, cnt, (const double *)S, (const double *)Y,
                (const double *)G, (double *)P);
  } else {
    SB_LB_CASES(two_loop_kernel, float, m, d, m, cnt, (const float *)S, (const float *)Y,
                (const float *)G, (float *)P);
  }
  SB_LAUNCH_CHECK();
  return SB_OK;
}

// ------------------------------------------------------------- state

size_t lbfgs_state_bytes(int dtype, int64_t B, int d, int m) {
  LbfgsBuffers b;
  b.dtype = dtype;
  b.B = B;
  b.d = d;
  b.m = m;
  Arena ar(nullptr, 0);
  lbfgs_carve(ar, b);
  return ar.off;
}

int lbfgs_carve(Arena &ar, LbfgsBuffers &b) {
  const size_t es = (b.dtype == DT_F64) ? 8 : 4;
  const int64_t B = b.B, d = b.d, m = b.m;
  auto take = [&](size_t n) -> void * { return (void *)ar.take<char>(n * es); };
  b.X = take(2 * B * d);
  b.G = take(2 * B * d);
  b.F = (void *)ar.take<double>(2 * B);
  b.Pd = take(B * d);
  b.S = take(B * m * d);
  b.Yh = take(B * m * d);
  b.rho = take(B * m);
  b.yy = take(B * m);
  b.alpha = take(B);
  b.gtp = take(B);
  b.cur = ar.take<int32_t>(B);
  b.head = ar.take<int32_t>(B);
  b.cnt = ar.take<int32_t>(B);
  b.iters = ar.take<int32_t>(B);
  b.ls = ar.take<int32_t>(B);
  b.status = ar.take<int32_t>(B);
  b.phase = ar.take<int32_t>(B);
  b.rowid = ar.take<int32_t>(B);
  b.active = ar.take<int32_t>(B);
  b.idx = ar.take<int32_t>(B);
  // (evaluations and active count side by side: one readback takes both)
  b.evals = ar.take<int64_t>(4);
  b.count = (int32_t *)(b.evals + 1);
  return ar.ok() ? SB_OK : SB_E_NOMEM;
}

template <typename T>
__global__ void lbfgs_init_kernel(int64_t B, int d, const T *X0, T *X, int32_t *cur,
                                  int32_t *head, int32_t *cnt, int32_t *iters, int32_t *ls,
                                  int32_t *status, int32_t *phase, int32_t *idx,
                                  int32_t *count, int64_t *evals) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t n = B * d;
  for (int64_t e = i; e < n; e += (int64_t)gridDim.x * blockDim.x) X[e] = X0[e];
  for (int64_t e = i; e < B; e += (int64_t)gridDim.x * blockDim.x) {
    cur[e] = 0;
    head[e] = 0;
    cnt[e] = 0;
    iters[e] = 0;
    ls[e] = 0;
    status[e] = ST_ACTIVE;
    phase[e] = PH_INIT;
    idx[e] = 0;
  }
  if (i == 0) {
    count[0] = 0;
    evals[0] = B;
  }
}

int launch_lbfgs_init(const LbfgsBuffers &b, const void *X0, hipStream_t s) {
  unsigned blocks = (unsigned)std::min<int64_t>(8192, ceil_div(b.B * b.d, 256));
  if (b.dtype == DT_F64)
    hipLaunchKernelGGL(lbfgs_init_kernel<double>, dim3(blocks), dim3(256), 0, s, b.B, b.d,
                       (const double *)X0, (double *)b.X, b.cur, b.head, b.cnt, b.iters, b.ls,
                       b.status, b.phase, b.idx, b.count, b.evals);
  else
    hipLaunchKernelGGL(lbfgs_init_kernel<float>, dim3(blocks), dim3(256), 0, s, b.B, b.d,
                       (const float *)X0, (float *)b.X, b.cur, b.head, b.cnt, b.iters, b.ls,
                       b.status, b.phase, b.idx, b.count, b.evals);
  SB_LAUNCH_CHECK();
  return SB_OK;
}

// Active starts' trial rows into idx[0, count).  Each wave ballots its
// starts and reserves its slice with one atomic: the order of the list
// depends on wave timing, the rows' results do not (every row of the
// contraction and of the epilogue is computed on its own).
__global__ __launch_bounds__(256) void compact_kernel(int64_t B, const int32_t *active,
                                                      const int32_t *rowid, int32_t *idx,
                                                      int32_t *count, int64_t *evals) {
  const int64_t s = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const bool on = s < B && active[s] != 0;
  const unsigned long long mask = __ballot(on);
  const int lane = threadIdx.x & 63;
  const int n = __popcll(mask);
  int base = 0;
  if (lane == 0 && n > 0) {
    base = atomicAdd(count, n);
    atomicAdd((unsigned long long *)evals, (unsigned long long)n);
  }
  base = __shfl(base, 0, 64);
  if (on) idx[base + __popcll(mask & ((1ull << lane) - 1ull))] = rowid[s];
}

// The step launch that precedes each compaction zeroes count.
int launch_compact(const LbfgsBuffers &b, hipStream_t s) {
  if (b.B > 0)
    hipLaunchKernelGGL(compact_kernel, dim3((unsigned)ceil_div(b.B, 256)), dim3(256), 0, s, b.B,
                       b.active, b.rowid, b.idx, b.count, b.evals);
  SB_LAUNCH_CHECK();
  return SB_OK;
}

template <typename T>
__global__ void lbfgs_gather_kernel(int64_t B, int d, const T *X, const T *G, const double *F,
                                    const int32_t *cur, const int32_t *st, const int32_t *its,
                                    T *Xo, void *lo, bool lo_f64, T *go, int32_t *sto,
                                    int32_t *ito) {
  const int64_t s = blockIdx.x;
  const int c = cur[s];
  for (int i = threadIdx.x; i < d; i += blockDim.x) {
    if (Xo) Xo[(size_t)s * d + i] = X[((size_t)c * B + s) * d + i];
    if (go) go[(size_t)s * d + i] = G[((size_t)c * B + s) * d + i];
  }
  if (threadIdx.x == 0) {
    if (lo) {
      if (lo_f64)
        ((double *)lo)[s] = F[(size_t)c * B + s];
      else
        ((T *)lo)[s] = (T)F[(size_t)c * B + s];
    }
    if (sto) sto[s] = st[s];
    if (ito) ito[s] = its[s];
  }
}

int launch_lbfgs_gather(const LbfgsBuffers &b, void *X, void *logl, bool logl_f64, void *grad,
                        int32_t *status, int32_t *iters, hipStream_t s) {
  if (b.B <= 0) return SB_OK;
  if (b.dtype == DT_F64)
    hipLaunchKernelGGL(lbfgs_gather_kernel<double>, dim3((unsigned)b.B), dim3(256), 0, s, b.B,
                       b.d, (const double *)b.X, (const double *)b.G, (const double *)b.F, b.cur,
                       b.status, b.iters, (double *)X, logl, logl_f64, (double *)grad, status,
                       iters);
  else
    hipLaunchKernelGGL(lbfgs_gather_kernel<float>, dim3((unsigned)b.B), dim3(256), 0, s, b.B, b.d,
                       (const float *)b.X, (const float *)b.G, (const double *)b.F, b.cur,
                       b.status, b.iters, (float *)X, logl, logl_f64, (float *)grad, status,
                       iters);
  SB_LAUNCH_CHECK();
  return SB_OK;
}

}  // namespace sb

// ====================================================================
// Batches: per-problem compaction, layout-preserving init and gather.
namespace sb {

// One workgroup per problem: active starts of [s0, s0 + B) in start order.
__global__ __launch_bounds__(1024) void compact_group_kernel(const BatchProb *probs,
                                                             const int32_t *active,
                                                             const int32_t *rowid,
                                                             const int64_t *rowoff, int32_t *idx,
                                                             int64_t *croff, int32_t *counts,
                                                             int64_t *evals) {
  __shared__ int32_t sc[1024];
  const BatchProb pr = probs[blockIdx.x];
  const int t = threadIdx.x;
  const int64_t B = pr.B, s0 = pr.s0;
  const int64_t per = (B + 1023) / 1024;
  const int64_t b0 = s0 + (int64_t)t * per, b1 = std::min<int64_t>(s0 + B, b0 + per);
  int32_t c = 0;
  for (int64_t i = b0; i < b1; ++i) c += active[i] ? 1 : 0;
  sc[t] = c;
  __syncthreads();
  for (int o = 1; o < 1024; o <<= 1) {
    int32_t v = (t >= o) ? sc[t - o] : 0;
    __syncthreads();
    sc[t] += v;
    __syncthreads();
  }
  int64_t pos = s0 + sc[t] - c;
  for (int64_t i = b0; i < b1; ++i)
    if (active[i]) {
      idx[pos] = rowid[i];
      croff[pos] = rowoff[i];
      ++pos;
    }
  if (t == 1023) {
    counts[blockIdx.x] = sc[1023];
    evals[blockIdx.x] += sc[1023];  // one workgroup per problem: no race
  }
}

int launch_compact_group(const BatchDev &b, const LbfgsBuffers &lb, int32_t *counts,
                         hipStream_t s) {
  hipLaunchKernelGGL(compact_group_kernel, dim3(b.n), dim3(1024), 0, s, b.probs, lb.active,
                     lb.rowid, lb.rowoff, lb.idx, lb.croff, counts, lb.pevals);
  SB_LAUNCH_CHECK();
  return SB_OK;
}

template <typename T>
__global__ void lbfgs_init_group_kernel(int64_t B, int64_t L, const T *X0, T *X, int32_t *cur,
                                        int32_t *head, int32_t *cnt, int32_t *iters, int32_t *ls,
                                        int32_t *status, int32_t *phase, int64_t *evals) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t e = i; e < L; e += stride) X[e] = X0[e];
  for (int64_t e = i; e < B; e += stride) {
    cur[e] = 0;
    head[e] = 0;
    cnt[e] = 0;
    iters[e] = 0;
    ls[e] = 0;
    status[e] = ST_ACTIVE;
    phase[e] = PH_INIT;
  }
  if (i == 0 && evals) evals[0] = B;
}

int launch_lbfgs_init_group(const LbfgsBuffers &b, const void *X0, hipStream_t s) {
  unsigned blocks = (unsigned)std::min<int64_t>(8192, ceil_div(std::max(b.Ltot, b.B), 256));
  if (b.dtype == DT_F64)
    hipLaunchKernelGGL(lbfgs_init_group_kernel<double>, dim3(blocks), dim3(256), 0, s, b.B,
                       b.Ltot, (const double *)X0, (double *)b.X, b.cur, b.head, b.cnt, b.iters,
                       b.ls, b.status, b.phase, b.evals);
  else
    hipLaunchKernelGGL(lbfgs_init_group_kernel<float>, dim3(blocks), dim3(256), 0, s, b.B,
                       b.Ltot, (const float *)X0, (float *)b.X, b.cur, b.head, b.cnt, b.iters,
                       b.ls, b.status, b.phase, b.evals);
  SB_LAUNCH_CHECK();
  return SB_OK;
}

template <typename T>
__global__ void lbfgs_gather_group_kernel(int64_t B, int64_t L, const int64_t *voff,
                                          const int32_t *vdim, const T *X, const double *F,
                                          const int32_t *cur, const int32_t *st, T *Xo,
                                          double *lo, int32_t *sto) {
  const int64_t s = blockIdx.x;
  const int c = cur[s];
  const int64_t vo = voff[s];
  for (int i = threadIdx.x; i < vdim[s]; i += blockDim.x) Xo[vo + i] = X[(size_t)c * L + vo + i];
  if (threadIdx.x == 0) {
    lo[s] = F[(size_t)c * B + s];
    sto[s] = st[s];
  }
}

int launch_lbfgs_gather_group(const LbfgsBuffers &b, void *X, double *logl, int32_t *status,
                              hipStream_t s) {
  if (b.B <= 0) return SB_OK;
  if (b.dtype == DT_F64)
    hipLaunchKernelGGL(lbfgs_gather_group_kernel<double>, dim3((unsigned)b.B), dim3(256), 0, s,
                       b.B, b.Ltot, b.voff, b.vdim, (const double *)b.X, (const double *)b.F,
                       b.cur, b.status, (double *)X, logl, status);
  else
    hipLaunchKernelGGL(lbfgs_gather_group_kernel<float>, dim3((unsigned)b.B), dim3(256), 0, s,
                       b.B, b.Ltot, b.voff, b.vdim, (const float *)b.X, (const double *)b.F,
                       b.cur, b.status, (float *)X, logl, status);
  SB_LAUNCH_CHECK();
  return SB_OK;
}

}  // namespace sb
