// Batched FP64 Cholesky factorisation, log-determinant and solves.
//
// H = L L^T (the whitening factor of the paper's appendix "Coordinate
// Whitening"); log det H = 2 sum_i log L_ii.  A failed pivot means H is not
// positive definite, i.e. the candidate is not a maximum (saddle filter of
// GreenDragon, generalised).
//
// Blocked right-looking factorisation with 64-wide panels, one or two launches per
// panel for every matrix of the batch, of one size or of their own.  What bounds a
// factorisation of few matrices is the chain of its panels, so there one launch does
// all of a panel at once: the workgroup of each trailing tile (I, J) solves the
// panel rows of I and J itself (L's 64 x 64 block by 16 x 16 blocks, their
// inverses and the products on the FP64 matrix cores) and subtracts X_I X_J^T;
// the workgroup of the first trailing tile goes on to factor it, the next
// panel's diagonal block.  Other workgroups still read the unsolved panel rows,
// so the solved ones go to the mirrored block of the upper triangle first and
// are moved by the next launch.  Where a panel has more tiles than the chip has CUs, a
// launch of its own solves its rows once, in place, and the tiles read them; the
// arithmetic and the results are the same.  n = 1024: 1 matrix 0.45 ms (27 us a panel
// where few tiles are left, of which the pivots take 16), 8 0.57, 64 1.71; three
// launches per panel (diagonal block, panel solve, trailing update, each element
// updated one column at a time) took 0.90, 1.09 and 2.40 ms.
#include <algorithm>

#include "internal.h"

namespace sb {

constexpr int NB = 64;

namespace {

typedef double d4v __attribute__((ext_vector_type(4)));

// The matrices of a batch: all n x n, one after another, or (nv) of size nv[c]
// at offset off[c], row-major with their size as leading dimension.
struct CholBatch {
  int n;
  const int32_t *nv;
  const int64_t *off;
  const double *A;  // first launch: the input (may be L)
  double *L;
  int32_t *info;
};
__device__ inline int chol_n(const CholBatch &b, int c) { return b.nv ? b.nv[c] : b.n; }
__device__ inline size_t chol_off(const CholBatch &b, int c) {
  return b.nv ? (size_t)b.off[c] : (size_t)c * b.n * b.n;
}

// 64 x 64 tiles in LDS: rows of 68 values, so that the 16 rows x 4 columns of
// an MFMA operand touch every bank evenly.
constexpr int LD = 68;
constexpr int LDD = 20;  // 16 x 16 inverses

__device__ inline d4v mfma(double a, double b, d4v c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
// LDS written by other lanes of this wave is visible after this
__device__ inline void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Column j of sub-block b by LDS and the library's root and division, a row per
// lane: for pivots that are not positive or near the ends of the exponent range.
__device__ __noinline__ int factor_columns_lds(double *T, int b) {
  const int lane = threadIdx.x;
  for (int j = 16 * b; j < 16 * b + 16; ++j) {
    const double p = T[j * LD + j];
    if (!uniform(p > 0.0)) return j + 1;
    const double d = sqrt(p), r = 1.0 / d;
    wave_lds_sync();
    if (lane >= j) T[lane * LD + j] = lane == j ? d : T[lane * LD + j] * r;
    wave_lds_sync();
    const double l = T[lane * LD + j];
    for (int k = j + 1; k < 16 * b + 16; ++k)
      if (lane >= k) T[lane * LD + k] -= l * T[k * LD + j];
    wave_lds_sync();
  }
  return 0;
}

// Factors the 64 x 64 block in T (lower triangle, rows from nb on the identity)
// in place, all four waves; returns 0 or the 1-based column of the first pivot
// that is not positive (the same in every thread).  Sixteen columns at a time:
// their update from the columns before on the matrix cores, then one wave with a
// row per lane and the 16 values in registers, so that the chain of pivots, which
// is what bounds a factorisation, needs no barrier.  A pivot's root comes from
// v_rsq_f64 and two Newton steps: r += r (1 - p r^2) / 2, then d = p r corrected by
// (p - d^2) r / 2.
__device__ int factor_block(double *T, int nb, int *fail_s) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lr = lane >> 4, lc = lane & 15;
  if (tid == 0) *fail_s = 0;
  for (int b = 0; 16 * b < nb; ++b) {
    if (b > 0 && wave >= b) {
      d4v acc = {0.0, 0.0, 0.0, 0.0};
      for (int kk = 0; kk < 16 * b; kk += 4)
        acc = mfma(T[(16 * wave + lc) * LD + kk + lr], T[(16 * b + lc) * LD + kk + lr], acc);
#pragma unroll
      for (int v = 0; v < 4; ++v) T[(16 * wave + lr + 4 * v) * LD + 16 * b + lc] -= acc[v];
    }
    __syncthreads();
    if (wave == 0) {
      double a[16];
#pragma unroll
      for (int k = 0; k < 16; ++k) a[k] = T[lane * LD + 16 * b + k];
      bool odd = false;
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const double p = wave_value(a[j], 16 * b + j);
        odd |= !(p > 0x1p-900 && p < 0x1p900);
        double r = __builtin_amdgcn_rsq(p);
        r = fma(0.5 * r, fma(-p * r, r, 1.0), r);
        r = fma(0.5 * r, fma(-p * r, r, 1.0), r);
        const double l = a[j] * r;
#pragma unroll
        for (int k = j + 1; k < 16; ++k) a[k] = fma(-l, wave_value(l, 16 * b + k), a[k]);
        const double d = p * r;
        a[j] = lane == 16 * b + j ? fma(0.5 * r, fma(-d, d, p), d) : l;
      }
      int f = 0;
      if (uniform(odd)) {
        f = factor_columns_lds(T, b);
      } else if (lane >= 16 * b) {
#pragma unroll
        for (int k = 0; k < 16; ++k) T[lane * LD + 16 * b + k] = a[k];
      }
      if (f && lane == 0) *fail_s = f;
    }
    __syncthreads();
    if (*fail_s) break;
  }
  return *fail_s;
}

// Factor in T (its first nb rows) to the matrix, zeros above the diagonal.
__device__ void put_block(const double *T, double *A, int n, int j0, int nb) {
  for (int e = threadIdx.x; e < NB * NB; e += 256) {
    const int i = e >> 6, k = e & 63;
    if (i < nb && k < nb) A[(size_t)(j0 + i) * n + j0 + k] = k <= i ? T[i * LD + k] : 0.0;
  }
}

// First launch: workgroup 0 of a matrix factors its first diagonal block, the
// others bring the rest of the lower triangle over and clear the upper one.
__global__ __launch_bounds__(256) void chol_first_kernel(CholBatch g) {
  __shared__ __attribute__((aligned(16))) double T[NB * LD];
  __shared__ int fail_s;
  const int c = blockIdx.x, n = chol_n(g, c);
  const size_t base = chol_off(g, c);
  const double *A = g.A + base;
  double *L = g.L + base;
  if (blockIdx.y > 0) {
    const int64_t total = (int64_t)n * n;
    for (int64_t e = (int64_t)(blockIdx.y - 1) * 256 + threadIdx.x; e < total;
         e += (int64_t)(gridDim.y - 1) * 256) {
      const int i = (int)(e / n), k = (int)(e - (int64_t)i * n);
      if (i < NB && k < NB) continue;
      if (k > i)
        L[e] = 0.0;
      else if (A != L)
        L[e] = A[e];
    }
    return;
  }
  const int nb = min(NB, n);
  for (int e = threadIdx.x; e < NB * NB; e += 256) {
    const int i = e >> 6, k = e & 63;
    T[i * LD + k] = (i < nb && k < nb) ? (k <= i ? A[(size_t)i * n + k] : 0.0)
                                       : (i == k ? 1.0 : 0.0);
  }
  __syncthreads();
  const int f = factor_block(T, nb, &fail_s);
  if (threadIdx.x == 0) g.info[c] = f;
  if (f)
    for (int e = threadIdx.x; e < NB * NB; e += 256) {  // (not factored: the input's triangle)
      const int i = e >> 6, k = e & 63;
      if (i < nb && k < nb) L[(size_t)i * n + k] = k <= i ? A[(size_t)i * n + k] : 0.0;
    }
  else
    put_block(T, L, n, 0, nb);
}

// Inverses of L_jj's diagonal 16 x 16 blocks (column lc per lane of wave `wave`'s
// block): as each x_k is known, its products leave the entries below.
__device__ __forceinline__ void invert_blocks(const double *Ls, double *Di) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, lr = lane >> 4, lc = lane & 15;
  const double *D = Ls + (16 * wave) * LD + 16 * wave;
  const double rp = 1.0 / D[lc * LD + lc];
  double x[16];
#pragma unroll
  for (int k = 0; k < 16; ++k) x[k] = k == lc ? 1.0 : 0.0;
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    x[k] *= wave_value(rp, k);
#pragma unroll
    for (int m = k + 1; m < 16; ++m) x[m] = fma(-D[m * LD + k], x[k], x[m]);
  }
  if (lr == 0)
#pragma unroll
    for (int k = 0; k < 16; ++k) Di[(16 * wave + k) * LDD + lc] = x[k];
}

// X = A L_jj^-T for this wave's 16 rows of I and (two) of J, 16 columns at a time:
// the rows in pi and pj, the results in XI and XJ.
__device__ __forceinline__ void solve_rows(const double *Ls, const double *Di, const d4v (&pi)[4],
                                           const d4v (&pj)[4], double *XI, double *XJ, bool two) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, lr = lane >> 4, lc = lane & 15;
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    const int row = 16 * wave + lc;
    d4v si = {0.0, 0.0, 0.0, 0.0}, sj = si;
#pragma unroll
    for (int kk = 0; kk < 16 * b; kk += 4) {
      const double l = Ls[(16 * b + lc) * LD + kk + lr];
      si = mfma(XI[row * LD + kk + lr], l, si);
      if (two) sj = mfma(XJ[row * LD + kk + lr], l, sj);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      XI[(16 * wave + lr + 4 * v) * LD + 16 * b + lc] = pi[b][v] - si[v];
      if (two) XJ[(16 * wave + lr + 4 * v) * LD + 16 * b + lc] = pj[b][v] - sj[v];
    }
    wave_lds_sync();
    d4v xi = {0.0, 0.0, 0.0, 0.0}, xj = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int kk = 0; kk < 16; kk += 4) {
      const double w = Di[(16 * b + lc) * LDD + kk + lr];
      xi = mfma(XI[row * LD + 16 * b + kk + lr], w, xi);
      if (two) xj = mfma(XJ[row * LD + 16 * b + kk + lr], w, xj);
    }
    wave_lds_sync();
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      XI[(16 * wave + lr + 4 * v) * LD + 16 * b + lc] = xi[v];
      if (two) XJ[(16 * wave + lr + 4 * v) * LD + 16 * b + lc] = xj[v];
    }
    wave_lds_sync();
  }
}

// This thread's 16 elements of a 64 x 64 tile in memory: row wave + 4 u, column lane.
template <class In>
__device__ __forceinline__ void tile_load(const double *A, int n, int i0, int j0, In in,
                                          double (&v)[16]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int u = 0; u < 16; ++u) {
    const int r = wave + 4 * u;
    v[u] = in(r, lane) ? A[(size_t)(i0 + r) * n + j0 + lane] : 0.0;
  }
}
__device__ __forceinline__ void tile_put(double *T, const double (&v)[16]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int u = 0; u < 16; ++u) T[(wave + 4 * u) * LD + lane] = v[u];
}
// This wave's 16 rows of a panel, item v of block b: row lr + 4 v, column 16 b + lc.
__device__ __forceinline__ void rows_load(const double *A, int n, int i0, int j0, bool on,
                                          d4v (&p)[4]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, lr = lane >> 4, lc = lane & 15;
#pragma unroll
  for (int b = 0; b < 4; ++b)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int r = 16 * wave + lr + 4 * v;
      p[b][v] = on && i0 + r < n ? A[(size_t)(i0 + r) * n + j0 + 16 * b + lc] : 0.0;
    }
}

// Panel p.  ONE: workgroups below `gt` (the tile count of the largest matrix) solve
// their panel rows and take a trailing tile each, the others move the solved rows of
// panel p - 1 into place.  Otherwise the panel rows are solved in place
// (chol_rows_kernel) and a workgroup takes its tile's from there.
template <bool ONE>
__global__ __launch_bounds__(256, ONE ? 1 : 2) void chol_panel_kernel(CholBatch g, int p, int gt) {
  __shared__ __attribute__((aligned(16))) double XI[NB * LD], XJ[NB * LD];
  __shared__ __attribute__((aligned(16))) double Lp[ONE ? NB * LD : 1];
  __shared__ double Di[ONE ? 4 * 16 * LDD : 1];  // inverses of L_jj's diagonal 16 x 16 blocks
  __shared__ int fail_s;
  double *Ls = ONE ? Lp : XJ;  // the next diagonal block (and with ONE L_jj's before it)
  const int c = blockIdx.y, n = chol_n(g, c), nblk = (n + NB - 1) / NB;
  double *A = g.L + chol_off(g, c);
  // A failed pivot stops its matrix at block q: panels before q are solved.
  // (Formed so that a failure noted while this launch runs, in block p + 1,
  // stops none of its workgroups.)
  const int inf = g.info[c], q = inf ? (inf - 1) / NB : nblk;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (ONE && (int)blockIdx.x >= gt) {
    const int I = p + (int)blockIdx.x - gt, pp = p - 1;
    if (pp < 0 || I >= nblk || pp >= q) return;
    const int i0 = I * NB, j0 = pp * NB, nr = min(NB, n - i0);
    // block (pp, I) of the upper triangle holds X_I transposed
    double v[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      const int r = wave + 4 * u;
      v[u] = lane < nr ? A[(size_t)(j0 + r) * n + i0 + lane] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < 16; ++u) XI[lane * LD + wave + 4 * u] = v[u];
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      const int r = wave + 4 * u;
      if (r < nr) A[(size_t)(i0 + r) * n + j0 + lane] = XI[r * LD + lane];
      if (lane < nr) A[(size_t)(j0 + r) * n + i0 + lane] = 0.0;
    }
    return;
  }
  const int T = nblk - 1 - p, t = blockIdx.x;
  if (T <= 0 || t >= T * (T + 1) / 2 || p >= q) return;
  // tile index -> (I, J) with I >= J
  int I = (int)((sqrtf(8.0f * (float)t + 1.0f) - 1.0f) * 0.5f);
  while ((I + 1) * (I + 2) / 2 <= t) ++I;
  while (I * (I + 1) / 2 > t) --I;
  const int J = t - I * (I + 1) / 2;
  const int j0 = p * NB, i0 = j0 + NB + I * NB, k0 = j0 + NB + J * NB;
  const int lr = lane >> 4, lc = lane & 15;
  const int wm = wave >> 1, wn = wave & 1;

  // Sums of products are formed from zero and subtracted once: rounded at their
  // own size and not at that of what they leave.  Every load first: the panel rows
  // of I and J (ONE: L_jj's block and this wave's 16 of each) and this wave's 32 x 32
  // quadrant of the tile (accumulator item v: row lr + 4 v, column lc)
  double lv[16], lw[16];
  d4v pi[4], pj[4], old[2][2], acc[2][2];
  if constexpr (ONE) {
    tile_load(A, n, j0, j0, [&](int r, int k) { return k <= r; }, lv);
    rows_load(A, n, i0, j0, true, pi);
    rows_load(A, n, k0, j0, I != J, pj);
  } else {
    tile_load(A, n, i0, j0, [&](int r, int) { return i0 + r < n; }, lv);
    if (I != J) tile_load(A, n, k0, j0, [&](int r, int) { return k0 + r < n; }, lw);
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int r = i0 + 32 * wm + 16 * i + lr + 4 * v, k = k0 + 32 * wn + 16 * j + lc;
        old[i][j][v] = (r < n && k <= r) ? A[(size_t)r * n + k] : 0.0;
        acc[i][j][v] = 0.0;
      }
  if constexpr (ONE) {
    tile_put(Ls, lv);
    __syncthreads();
    invert_blocks(Ls, Di);
    __syncthreads();
    solve_rows(Ls, Di, pi, pj, XI, XJ, I != J);
  } else {
    tile_put(XI, lv);
    if (I != J) tile_put(XJ, lw);
  }
  __syncthreads();
  const double *B = I != J ? XJ : XI;
  if (I != J || wm >= wn) {  // (a diagonal tile's upper quadrant is not kept)
#pragma unroll 4
    for (int kk = 0; kk < NB; kk += 4) {
      double af[2], bf[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        af[i] = XI[(32 * wm + 16 * i + lc) * LD + kk + lr];
        bf[i] = B[(32 * wn + 16 * i + lc) * LD + kk + lr];
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = mfma(af[i], bf[j], acc[i][j]);
    }
  }
  if (ONE && I == J)  // the solved rows, transposed into block (p, I) of the upper triangle
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      const int r = wave + 4 * u;
      if (i0 + lane < n) A[(size_t)(j0 + r) * n + i0 + lane] = XI[lane * LD + r];
    }
  if (t > 0) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int r = i0 + 32 * wm + 16 * i + lr + 4 * v, k = k0 + 32 * wn + 16 * j + lc;
          if (r < n && k <= r) A[(size_t)r * n + k] = old[i][j][v] - acc[i][j][v];
        }
    return;
  }
  // the next diagonal block (Ls is free: tile 0 is a diagonal one, without XJ, and
  // with ONE every wave has passed its products with L_jj's block)
  const int nb = min(NB, n - i0);
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int r = 32 * wm + 16 * i + lr + 4 * v, k = 32 * wn + 16 * j + lc;
        Ls[r * LD + k] = (r < nb && k < nb) ? old[i][j][v] - acc[i][j][v] : (r == k ? 1.0 : 0.0);
      }
  __syncthreads();
  const int f = factor_block(Ls, nb, &fail_s);
  if (f) {
    if (tid == 0) g.info[c] = i0 + f;
    return;
  }
  put_block(Ls, A, n, i0, nb);
}

// The rows of panel p solved in place, 64 of them a workgroup.
__global__ __launch_bounds__(256, 2) void chol_rows_kernel(CholBatch g, int p) {
  __shared__ __attribute__((aligned(16))) double Ls[NB * LD], XI[NB * LD];
  __shared__ double Di[4 * 16 * LDD];
  const int c = blockIdx.y, n = chol_n(g, c), nblk = (n + NB - 1) / NB;
  double *A = g.L + chol_off(g, c);
  const int inf = g.info[c], q = inf ? (inf - 1) / NB : nblk;
  const int I = p + 1 + blockIdx.x, i0 = I * NB, j0 = p * NB;
  if (I >= nblk || p >= q) return;
  double lv[16];
  d4v pi[4];
  tile_load(A, n, j0, j0, [&](int r, int k) { return k <= r; }, lv);
  rows_load(A, n, i0, j0, true, pi);
  tile_put(Ls, lv);
  __syncthreads();
  invert_blocks(Ls, Di);
  __syncthreads();
  solve_rows(Ls, Di, pi, pi, XI, nullptr, false);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int u = 0; u < 16; ++u) {  // (this wave's own rows)
    const int r = 16 * wave + u;
    if (i0 + r < n) A[(size_t)(i0 + r) * n + j0 + lane] = XI[r * LD + lane];
  }
}

int chol_run(int C, int n_max, const CholBatch &g, hipStream_t s) {
  const int64_t total = (int64_t)n_max * n_max;
  const unsigned copies =
      n_max > NB ? (unsigned)std::min<int64_t>(512, ceil_div(total, 2048)) : 0u;
  hipLaunchKernelGGL(chol_first_kernel, dim3(C, 1 + copies), dim3(256), 0, s, g);
  SB_LAUNCH_CHECK();
  const int nblk = (int)ceil_div(n_max, NB);
  if (nblk < 2) return SB_OK;
  bool mirrored = false;  // panel p - 1's rows are still in the upper triangle
  for (int p = 0; p < nblk; ++p) {
    const int T = nblk - 1 - p, gt = T * (T + 1) / 2;
    const int moves = mirrored ? nblk - p : 0;  // rows of blocks p .. of panel p - 1
    // More tiles than CUs: a tile's workgroup that solves its panel rows itself has
    // a CU's LDS alone, so a second round of them costs more than the launch that
    // solves each row once (us, one launch a panel : two): n = 512, 8 matrices (224
    // tiles in the first panel) 244 : 255, 16 (448) 285 : 266, 512 3946 : 2029; n =
    // 320, 16 (160) 155 : 159, 32 (320) 174 : 165; n = 2048, 64 21579 : 9041.
    if ((int64_t)C * gt > 256) {
      hipLaunchKernelGGL(chol_rows_kernel, dim3((unsigned)T, C), dim3(256), 0, s, g, p);
      SB_LAUNCH_CHECK();
      hipLaunchKernelGGL(chol_panel_kernel<false>, dim3((unsigned)gt, C), dim3(256), 0, s, g, p,
                         gt);
      SB_LAUNCH_CHECK();
      continue;
    }
    if (gt + moves == 0) break;
    hipLaunchKernelGGL(chol_panel_kernel<true>, dim3((unsigned)(gt + moves), C), dim3(256), 0, s, g,
                       p, gt);
    SB_LAUNCH_CHECK();
    mirrored = true;
  }
  return SB_OK;
}

}  // namespace

int chol_batched(int C, int n, const double *A, double *L, int32_t *info, hipStream_t s) {
  if (C <= 0 || n <= 0) return SB_OK;
  return chol_run(C, n, CholBatch{n, nullptr, nullptr, A, L, info}, s);
}

// In-place factorisation of C matrices of sizes nv[c] at offsets off[c].
int chol_batched_u(int C, const int32_t *nv, const int64_t *off, int n_max, double *L,
                   int32_t *info, hipStream_t s) {
  if (C <= 0 || n_max <= 0) return SB_OK;
  return chol_run(C, n_max, CholBatch{0, nv, off, L, L, info}, s);
}

// log det = 2 sum_i log L_ii from the factor (fixed-order reduction), NaN if it failed.
__global__ __launch_bounds__(256) void logdet_kernel(int n, const double *L,
                                                     const int32_t *info, double *logdet) {
  const int c = blockIdx.x;
  __shared__ double red[4];
  double v = 0.0;
  for (int i = threadIdx.x; i < n; i += 256) v += log(L[(size_t)c * n * n + (size_t)i * n + i]);
  v = block_sum<256>(v, red);
  if (threadIdx.x == 0) logdet[c] = info[c] ? NAN : 2.0 * v;
}

int launch_logdet(int C, int n, const double *L, const int32_t *info, double *logdet,
                  hipStream_t s) {
  if (C <= 0) return SB_OK;
  hipLaunchKernelGGL(logdet_kernel, dim3(C), dim3(256), 0, s, n, L, info, logdet);
  SB_LAUNCH_CHECK();
  return SB_OK;
}

// Solve L L^T x = b, one workgroup of 16 waves per matrix, x in LDS, 64 rows at
// a time forward (L z = b) and back (L^T x = z).  One wave carries the chain: it
// adds the block's product with the block solved last and substitutes through
// the diagonal block, both from LDS.  Meanwhile the others sum the next block's
// products with everything solved before that and bring its two tiles in, so
// that reading L, which is what bounds the solve (one workgroup takes about a
// hundredth of the memory rate), goes on all the time.  n = 1024: 350 -> 235 us.
constexpr int SV_T = 1024, SV_W = SV_T / 64 - 1;  // (15 waves beside the chain)
constexpr int SV_LD = 65;
__global__ __launch_bounds__(SV_T) void chol_solve_kernel(CholBatch g, const double *ball,
                                                          double *xall, int64_t vs,
                                                          const int32_t *info) {
  extern __shared__ double xs[];  // [n]
  __shared__ double TD[NB * SV_LD], TL[NB * SV_LD];  // diagonal block, its neighbour
  __shared__ double part[2][SV_W][64];
  const int c = blockIdx.x, n = chol_n(g, c), nblk = (n + NB - 1) / NB;
  const double *L = g.L + chol_off(g, c);
  const double *b = ball + (size_t)c * vs;
  double *x = xall + (size_t)c * vs;
  const int tid = threadIdx.x, lane = tid & 63, w = uniform(tid >> 6);
  if (info && info[c] != 0) {
    for (int i = tid; i < n; i += SV_T) x[i] = NAN;
    return;
  }
  for (int i = tid; i < n; i += SV_T) xs[i] = b[i];
  // tile (bi, bj) through the registers of the 15 waves (zeros outside L)
  constexpr int NE = (NB * NB + 64 * SV_W - 1) / (64 * SV_W);
  auto fetch = [&](int bi, int bj, double (&v)[NE]) {
#pragma unroll
    for (int q = 0; q < NE; ++q) {
      const int e = tid - 64 + 64 * SV_W * q, i = bi * NB + (e >> 6), k = bj * NB + (e & 63);
      v[q] = (e < NB * NB && i < n && k <= i) ? L[(size_t)i * n + k] : 0.0;
    }
  };
  auto put = [&](double *T, const double (&v)[NE]) {
#pragma unroll
    for (int q = 0; q < NE; ++q) {
      const int e = tid - 64 + 64 * SV_W * q;
      if (e < NB * NB) T[(e >> 6) * SV_LD + (e & 63)] = v[q];
    }
  };
  if (w > 0) {
    double v[NE];
    fetch(0, 0, v);
    put(TD, v);
  }
  __syncthreads();
  for (int i = 0; i < nblk; ++i) {
    const int i0 = i * NB, nb = min(NB, n - i0), pb = i & 1;
    double vl[NE], vd[NE];
    if (w == 0) {
      double t = i > 1 ? part[pb][0][lane] : 0.0;
      if (i > 0)
#pragma unroll 16
        for (int k = 0; k < NB; ++k) t += TL[lane * SV_LD + k] * xs[i0 - NB + k];
      double val = lane < nb ? xs[i0 + lane] - t : 0.0;
      const double rp = lane < nb ? 1.0 / TD[lane * SV_LD + lane] : 1.0;
#pragma unroll 8
      for (int cc = 0; cc < nb; ++cc) {  // (unrolled: the reads of TD leave the chain)
        const double xc = wave_value(val * rp, cc);
        if (lane == cc) val = xc;
        if (lane > cc) val -= TD[lane * SV_LD + cc] * xc;
      }
      if (lane < nb) xs[i0 + lane] = val;
    } else if (i + 1 < nblk) {
      fetch(i + 1, i, vl);
      fetch(i + 1, i + 1, vd);
      // rows w - 1 + 15 q of block i + 1 with the solved k < i0, lanes split k
      constexpr int NR = (NB + SV_W - 1) / SV_W;
      double acc[NR];
      const double *Lr[NR];
#pragma unroll
      for (int q = 0; q < NR; ++q) {
        const int r = w - 1 + SV_W * q, row = i0 + NB + r;
        acc[q] = 0.0;
        Lr[q] = L + (size_t)(r < NB && row < n ? row : 0) * n;  // (others: sums not used)
      }
      int k = lane;
      for (; k + 64 * 3 < i0; k += 64 * 4) {
        double lv[4][NR];
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int q = 0; q < NR; ++q) lv[u][q] = Lr[q][k + 64 * u];
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int q = 0; q < NR; ++q) acc[q] += lv[u][q] * xs[k + 64 * u];
      }
      for (; k < i0; k += 64)
#pragma unroll
        for (int q = 0; q < NR; ++q) acc[q] += Lr[q][k] * xs[k];
#pragma unroll
      for (int q = 0; q < NR; ++q) {
        const double t = wave_sum(acc[q]);
        if (lane == 0 && w - 1 + SV_W * q < NB) part[pb ^ 1][0][w - 1 + SV_W * q] = t;
      }
    }
    __syncthreads();
    if (w > 0 && i + 1 < nblk) {
      put(TL, vl);
      put(TD, vd);
    }
    __syncthreads();
  }
  for (int i = nblk - 1; i >= 0; --i) {
    const int i0 = i * NB, nb = min(NB, n - i0), pb = i & 1;
    double vl[NE], vd[NE];
    if (w == 0) {
      double t = 0.0;
      if (i + 2 < nblk)
#pragma unroll
        for (int u = 0; u < SV_W; ++u) t += part[pb][u][lane];
      if (i + 1 < nblk) {
        const int nn = min(NB, n - i0 - NB);  // (rows past the matrix: zeros in TL)
#pragma unroll 16
        for (int k = 0; k < nn; ++k) t += TL[k * SV_LD + lane] * xs[i0 + NB + k];
      }
      double val = lane < nb ? xs[i0 + lane] - t : 0.0;
      const double rp = lane < nb ? 1.0 / TD[lane * SV_LD + lane] : 1.0;
#pragma unroll 8
      for (int cc = nb - 1; cc >= 0; --cc) {
        const double xc = wave_value(val * rp, cc);
        if (lane == cc) val = xc;
        if (lane < cc) val -= TD[cc * SV_LD + lane] * xc;
      }
      if (lane < nb) xs[i0 + lane] = val;
    } else if (i > 0) {
      fetch(i, i - 1, vl);
      fetch(i - 1, i - 1, vd);
      // column lane of block i - 1 with the solved rows k >= i0 + 64, waves split k
      const double *Lc = L + i0 - NB + lane;
      double acc = 0.0;
      int k = i0 + NB + w - 1;
      for (; k + SV_W * 15 < n; k += SV_W * 16) {
        double lv[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) lv[u] = Lc[(size_t)(k + SV_W * u) * n];
#pragma unroll
        for (int u = 0; u < 16; ++u) acc += lv[u] * xs[k + SV_W * u];
      }
      for (; k < n; k += SV_W) acc += Lc[(size_t)k * n] * xs[k];
      part[pb ^ 1][w - 1][lane] = acc;
    }
    __syncthreads();
    if (w > 0 && i > 0) {
      put(TL, vl);
      put(TD, vd);
    }
    __syncthreads();
  }
  for (int i = tid; i < n; i += SV_T) x[i] = xs[i];
}

static int solve_run(int C, int n_max, const CholBatch &g, const double *b, double *x, int64_t vs,
                     const int32_t *info, hipStream_t s) {
  if (C <= 0) return SB_OK;
  const size_t shm = sizeof(double) * (size_t)n_max;
  if (shm > 64 * 1024) {
    set_error("solve dimension %d too large", n_max);
    return SB_E_UNSUPPORTED;
  }
  hipLaunchKernelGGL(chol_solve_kernel, dim3(C), dim3(SV_T), shm, s, g, b, x, vs, info);
  SB_LAUNCH_CHECK();
  return SB_OK;
}

int launch_chol_solve(int C, int n, const double *L, const double *b, double *x,
                      const int32_t *info, hipStream_t s) {
  return solve_run(C, n, CholBatch{n, nullptr, nullptr, nullptr, (double *)L, nullptr}, b, x, n,
                   info, s);
}

// Matrix c of size nv[c] at offset off[c]; its rows of b and x start at c * vs.
int launch_chol_solve_u(int C, const int32_t *nv, const int64_t *off, int n_max, const double *L,
                        const double *b, double *x, int64_t vs, const int32_t *info,
                        hipStream_t s) {
  return solve_run(C, n_max, CholBatch{0, nv, off, nullptr, (double *)L, nullptr}, b, x, vs, info,
                   s);
}

}  // namespace sb

// ====================================================================
// Uneven batches: matrix c has size n[c] and starts at off[c] (row-major,
// leading dimension n[c]); vectors of matrix c start at voff[c].
namespace sb {

__global__ __launch_bounds__(256) void logdet_u_kernel(const int32_t *nv, const int64_t *off,
                                                       const double *L, const int32_t *info,
                                                       double *logdet) {
  const int c = blockIdx.x;
  const int n = nv[c];
  __shared__ double red[4];
  double v = 0.0;
  for (int i = threadIdx.x; i < n; i += 256) v += log(L[off[c] + (size_t)i * n + i]);
  v = block_sum<256>(v, red);
  if (threadIdx.x == 0) logdet[c] = info[c] ? NAN : 2.0 * v;
}

int launch_logdet_u(int C, const int32_t *nv, const int64_t *off, const double *L,
                    const int32_t *info, double *logdet, hipStream_t s) {
  if (C <= 0) return SB_OK;
  hipLaunchKernelGGL(logdet_u_kernel, dim3(C), dim3(256), 0, s, nv, off, L, info, logdet);
  SB_LAUNCH_CHECK();
  return SB_OK;
}

}  // namespace sb
