// The FP64 evaluation of 16 points by one workgroup: contraction on the matrix
// cores, the family's l and the gradient, with everything between them in LDS.
// Shared by the fused evaluation launch and by the small-problem optimiser,
// which runs it between its steps.
#pragma once

#include "internal.h"
#include "mixture.h"

namespace sb {

namespace fused {

typedef double d2v __attribute__((ext_vector_type(2)));
typedef double d4v __attribute__((ext_vector_type(4)));

constexpr int kRows = 16;  // points per tile

// LDS bytes of a tile.
inline size_t lds_bytes(int K, int dp) {
  return 8 * ((size_t)K * kRows * (dp + 2) + (size_t)kRows * K * (dp / 16) + (size_t)kRows * K +
              (size_t)K * dp);
}

// NT threads; NS 16-column blocks per wave, every wave running all NS (a wave
// whose last slot lies past the K x dp outputs multiplies block 0 again and
// keeps nothing of it), so that the slot loops hold no branch and each slot's
// loads wait only for their own data.  FAST: d is a multiple of 8 and P is
// 16-byte aligned (the B loads below).  Rows: src(i[], row[]) the operand rows
// of tile rows i (-1: none, evaluated as zeros), dst(i) the output row of tile
// row i (-1: none), aux(i) its row of aux.  new_mu: MU is staged (a tile that
// follows another in the same LDS has it).  tid: threadIdx.x.  X, l and the gradient are FP64.
template <int NT, int NS, bool FAST, class Rows>
__device__ __forceinline__ void tile(const Model &m, int dp, const double *X, int64_t ldx,
                                     const Rows &rows, double *logl, double *grad, int64_t ldg,
                                     double *aux, double *lds, bool new_mu, const int tid) {
  constexpr int R = kRows, NW = NT / 64;
  static_assert(NT >= 16 * R, "the mixture row epilogue maps 16 rows onto 256 threads");
  const int d = m.d, K = m.K, nbk = dp / 16, nb = K * nbk;
  // D rows padded by 16 bytes: the 16 rows of a fragment read start on
  // different banks (a row of dp doubles is a multiple of the bank width)
  const int ld = dp + 2;
  const int lane = tid & 63, wave = tid >> 6;
  // LDS: D[k][i][j] = delta_k of row i (zero past d and past M), then
  // delta_k * Y_k, then the weighted Y; qs[i][k][t] the q partial of row i, component k, column
  // block t; sc[i][k] the row's gradient weights; MU[k][j] = mu_k
  double *D = lds;
  double *qs = D + (size_t)K * R * ld;
  double *sc = qs + R * K * nbk;
  double *MU = sc + R * K;  // mu_k, zero past d: [K][dp]
  // beta_k of the mixture row epilogue's lane k = tid % 16 (index clamped,
  // K >= 1), loaded here so that it arrives with the staging's values
  const double beta_k = m.beta[(tid & 15) < K ? (tid & 15) : 0];
  // blocks b = wave + NW s: column block t = b / K of component k = b % K
  const int fr = lane & 15, fg = lane >> 4;
  d4v acc[NS];
  int bk[NS], bn[NS];
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    acc[s] = d4v{0.0, 0.0, 0.0, 0.0};
    const int b = wave + NW * s;
    bk[s] = b < nb ? b % K : 0;
    bn[s] = b < nb ? (b / K) * 16 : 0;
  }
  // k in groups of 32: in group g lane l holds the 8 consecutive values j =
  // 32 g + 8 (l / 16) + u, u < 8, of its B row (n = bn + l % 16 of P_k) and
  // of its A row, and MFMA u of the group takes them (each MFMA sums four
  // k values 8 apart; every k of the group exactly once).  A lane's B values
  // are two full 32-byte runs of one row, 16 rows per load: whole cache
  // lines.  Slot s's values of group g + 1 load as soon as its MFMAs of
  // group g have read them, so they fly while the other slots multiply.
  // With FAST a lane's 8 values lie in its row or wholly past it: the loads
  // are unconditional, from row 0 when past d, and the values are zeroed
  // where the MFMAs take them (bin), not where they land, so that no wait
  // follows the loads.
  bool bin[NS];
  auto bload = [&](int s, int g, d2v (&bv)[4]) {
    const int n = bn[s] + fr, j0 = 32 * g + 8 * fg;
    if constexpr (FAST) {
      const bool in = n < d && j0 < d;
      const double *p = m.P64 + ((size_t)bk[s] * d + (in ? n : 0)) * d + (in ? j0 : 0);
#pragma unroll
      for (int u = 0; u < 4; ++u) bv[u] = *(const d2v *)(p + 2 * u);
      bin[s] = in;
    } else {
      const double *p = m.P64 + ((size_t)bk[s] * d + n) * d + j0;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const bool i0 = n < d && j0 + 2 * u < d, i1 = n < d && j0 + 2 * u + 1 < d;
        bv[u] = d2v{i0 ? p[2 * u] : 0.0, i1 ? p[2 * u + 1] : 0.0};
      }
      bin[s] = true;
    }
  };
  // the first k-group's P values load before the staging below, so that
  // the two round trips overlap
  d2v bb[NS][4];
#pragma unroll
  for (int s = 0; s < NS; ++s) bload(s, 0, bb[s]);

  // Staging: every global load of the tile (mu, the row map, x) is issued
  // before the first one is used, so the tile waits for one or two round
  // trips rather than one per value.  Values go in pairs (j, j + 1): a
  // thread takes at most kPairs pairs of x (R dp / 2 <= 1024 for dp <= 128)
  // and one pair of mu (K dp / 2 <= 192).
  constexpr int kPairs = 1024 / NT;
  const int hp = dp / 2, np = R * hp;
  const int mk = new_mu && tid < K * hp ? tid / hp : -1, mj = 2 * (tid % hp);
  double mv0 = 0.0, mv1 = 0.0;
  if (mk >= 0) {
    const double *p = m.mu64 + (size_t)mk * d + mj;
    if (mj < d) mv0 = p[0];
    if (mj + 1 < d) mv1 = p[1];
  }
  int ti[kPairs];
  int64_t src[kPairs];
#pragma unroll
  for (int u = 0; u < kPairs; ++u) ti[u] = (tid + NT * u) / hp;
  rows.src(ti, src);
#pragma unroll
  for (int u = 0; u < kPairs; ++u)
    if (tid + NT * u >= np) src[u] = -1;
  d2v xv[kPairs];
#pragma unroll
  for (int u = 0; u < kPairs; ++u) {
    const int j = 2 * ((tid + NT * u) % hp);
    const double *p = X + src[u] * ldx + j;
    xv[u] = d2v{src[u] >= 0 && j < d ? p[0] : 0.0, src[u] >= 0 && j + 1 < d ? p[1] : 0.0};
  }
  if (mk >= 0) *(d2v *)&MU[mk * dp + mj] = d2v{mv0, mv1};
  __syncthreads();
  // D[k][i][j] = delta_k of row i (zero past d and past M)
#pragma unroll
  for (int u = 0; u < kPairs; ++u) {
    const int e = tid + NT * u;
    if (e < np) {
      const int i = e / hp, j = 2 * (e % hp);
      for (int k = 0; k < K; ++k)
        *(d2v *)&D[((size_t)k * R + i) * ld + j] =
            src[u] >= 0 ? xv[u] - *(const d2v *)&MU[k * dp + j] : d2v{0.0, 0.0};
    }
  }
  __syncthreads();

  const int ng = dp / 32;
  for (int g = 0; g < ng; ++g) {
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const double *ar = &D[((size_t)bk[s] * R + fr) * ld + 32 * g + 8 * fg];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const d2v av = *(const d2v *)(ar + 2 * u);
        const d2v bv = bin[s] ? bb[s][u] : d2v{0.0, 0.0};
        acc[s] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[0], bv[0], acc[s], 0, 0, 0);
        acc[s] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[1], bv[1], acc[s], 0, 0, 0);
      }
      if (g + 1 < ng) bload(s, g + 1, bb[s]);
    }
  }

  // q partials: item v of lane l is Y_k[row fg + 4 v][column bn + fr];
  // once every wave is done reading D as the A operand, each item's product
  // delta_k * Y_k replaces its delta in D, and qs[i][k][t] sums block t's 16
  // products of row i in column order (threads along rows: the rows' 8-byte
  // reads fall on different banks)
  __syncthreads();
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    if (wave + NW * s < nb) {
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        double *t = &D[((size_t)bk[s] * R + fg + 4 * v) * ld + bn[s] + fr];
        *t = *t * acc[s][v];
      }
    }
  }
  __syncthreads();
  for (int e = tid; e < R * K * nbk; e += NT) {
    const int i = e % R, k = (e / R) % K, t = e / (R * K);
    const double *p = &D[((size_t)k * R + i) * ld + 16 * t];
    double q = 0.0;
#pragma unroll
    for (int c = 0; c < 16; ++c) q += p[c];
    qs[(i * K + k) * nbk + t] = q;
  }
  __syncthreads();

  // per row: l, the responsibilities (or the Student-t weight) in FP64
  if (m.family == SB_FAMILY_STUDENT_T) {
    if (tid < R) {
      const int i = tid;
      const int64_t orow = rows.dst(i);
      if (orow >= 0) {
        const double *qp = qs + (size_t)i * K * nbk;
        double q = 0;
        for (int t = 0; t < nbk; ++t) q += qp[t];
        const double nd = m.nu + (double)d;
        logl[orow] = m.c + m.beta[0] - 0.5 * nd * log1p(q / m.nu);
        if (aux) aux[rows.aux(i) * K] = q;
        sc[i * K] = nd / (m.nu + q);
      }
    }
  } else if (tid < 256) {
    // 16 lanes per row (16 rows of 16: the first four waves), component k in
    // lane k (K <= 12 here): a_k = beta_k - q_k / 2, the wave maximum, each
    // exp(a_k - max) formed once in its lane and the K of them added in
    // component order from zero, lse = max + log(sum) (a_0 when K = 1),
    // r_k = exp(a_k - lse): the arithmetic and order of the row epilogue
    // of the two-launch path
    const int i = tid >> 4, k = tid & 15, base = (tid & 63) & ~15;
    double a = -INFINITY;
    if (k < K) {
      const double *qp = qs + ((size_t)i * K + k) * nbk;
      double q = 0;
      for (int t = 0; t < nbk; ++t) q += qp[t];
      a = beta_k - 0.5 * q;
    }
    double mx = a;
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) mx = fmax(mx, __shfl_xor(mx, o, 64));
    double lse;
    if (K == 1) {
      lse = __shfl(a, base, 64);
    } else {
      const double e = k < K ? exp(a - mx) : 0.0;
      double ssum = 0;
      for (int c = 0; c < K; ++c) ssum += __shfl(e, base + c, 64);
      lse = mx + log(ssum);
    }
    const int64_t orow = rows.dst(i);
    if (orow >= 0 && k < K) {
      const double r = K == 1 ? 1.0 : exp(a - lse);
      sc[i * K + k] = r;
      if (aux) aux[rows.aux(i) * K + k] = r;
      if (k == 0) logl[orow] = m.c + lse;
    }
  }
  if (!grad) return;
  __syncthreads();  // (also: every wave is done reading D)
  // D <- weight_k * Y_k (a component of weight zero adds nothing, as in the
  // two-launch path)
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    if (wave + NW * s < nb) {
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int i = fg + 4 * v;
        const double w = sc[i * K + bk[s]];
        D[((size_t)bk[s] * R + i) * ld + bn[s] + fr] = w != 0.0 ? w * acc[s][v] : 0.0;
      }
    }
  }
  __syncthreads();
  // grad = -sum_k D_k, components in order, 16-byte stores where aligned
  for (int e = tid; e < R * (dp / 2); e += NT) {
    const int i = e / (dp / 2), j = 2 * (e % (dp / 2));
    const int64_t orow = rows.dst(i);
    if (orow < 0 || j >= d) continue;
    d2v s = d2v{0.0, 0.0};
    for (int k = 0; k < K; ++k) s += *(const d2v *)&D[((size_t)k * R + i) * ld + j];
    double *go = grad + orow * ldg + j;
    if (j + 1 < d && (((uintptr_t)go) & 15) == 0) {
      *(d2v *)go = -s;
    } else {
      go[0] = -s[0];
      if (j + 1 < d) go[1] = -s[1];
    }
  }
}

}  // namespace fused

}  // namespace sb
