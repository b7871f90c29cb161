// Fused FP64 log-likelihood and gradient for small dimensions (step A3 with
// its row epilogue in one launch).
//
// One workgroup takes 16 points and every component: it stages
// delta_k = x - mu_k of its rows in LDS, multiplies them by P_k on the FP64
// matrix cores (16x16x4 MFMAs, each wave owning a set of 16-column blocks of
// the K x d outputs, P read straight from the L2), forms q_k = delta_k . Y_k
// per row, the family's l, and the gradient -sum_k r_k Y_k (mixture) or
// -((nu + d)/(nu + q)) Y (Student-t) through the same LDS, and writes l and
// the gradient once.  Y and the q partials never go to HBM, and the two
// launches of the GEMM + epilogue path become one: at d <= 128 the path is
// bound by latency and launch count rather than by the matrix cores.
//
// The k index of the contraction is taken in groups of 32, each lane holding
// 8 consecutive values of its A and B rows (any order of the j sum is the
// same sum in exact arithmetic; in FP64 the rounding differs from the GEMM
// path's by a few ulps).
#include <cstdlib>

#include "fused_tile.h"
#include "internal.h"

namespace sb {

namespace {

constexpr int kMaxSlots = 6;   // 16-column blocks per wave (K * dp <= 384)

struct FusedArgs {
  Model m;
  ASrc a;                       // kind 0: rows of X (FP64), optional row map
  int64_t M;
  const int32_t *count;         // device row count (nullable -> M)
  const int32_t *outmap;        // output row of each row (nullable)
  double *logl;
  double *grad;                 // [*][ldg] (nullable)
  int64_t ldg;
  double *aux;                  // [M][K]: responsibilities / q (nullable)
  int dp;                       // d rounded up to a multiple of 32
};

// Rows r0 .. r0 + 15 of the M rows of a launch, operand and output rows through
// optional maps.
struct MapRows {
  int64_t r0, M;
  const int32_t *rowmap, *outmap;
  template <int N>
  __device__ __forceinline__ void src(const int (&i)[N], int64_t (&row)[N]) const {
    // (the map is read at a clamped row, without a branch, so its loads issue together)
#pragma unroll
    for (int u = 0; u < N; ++u) row[u] = r0 + i[u] < M ? r0 + i[u] : M - 1;
    if (rowmap) {
#pragma unroll
      for (int u = 0; u < N; ++u) row[u] = rowmap[row[u]];
    }
#pragma unroll
    for (int u = 0; u < N; ++u)
      if (r0 + i[u] >= M) row[u] = -1;
  }
  __device__ __forceinline__ int64_t dst(int i) const {
    const int64_t row = r0 + i;
    if (row >= M) return -1;
    return outmap ? (int64_t)outmap[row] : row;
  }
  __device__ __forceinline__ int64_t aux(int i) const { return r0 + i; }
};

template <int NS, bool FAST>
__global__ __launch_bounds__(256) void fused_logl_grad_kernel(FusedArgs f) {
  extern __shared__ __attribute__((aligned(16))) double lds[];
  const int64_t M = f.count ? (int64_t)(*f.count) : f.M;
  const int64_t r0 = (int64_t)blockIdx.x * fused::kRows;
  if (r0 >= M) return;
  const MapRows rows{r0, M, f.a.rowmap, f.outmap};
  fused::tile<256, NS, FAST>(f.m, f.dp, (const double *)f.a.X, f.a.ldx, rows, f.logl, f.grad, f.ldg,
                             f.aux, lds, true, threadIdx.x);
}

template <int NS>
void launch_fused(bool fast, dim3 grid, size_t lds, hipStream_t s, const FusedArgs &f) {
  if (fast)
    hipLaunchKernelGGL((fused_logl_grad_kernel<NS, true>), grid, dim3(256), lds, s, f);
  else
    hipLaunchKernelGGL((fused_logl_grad_kernel<NS, false>), grid, dim3(256), lds, s, f);
}

}  // namespace

bool fused_logl_grad_ok(const Model &m, const ASrc &a) {
  const char *e = getenv("SB_FUSED");  // "0": the two-launch path (for comparison)
  if (e && e[0] == '0') return false;
  // d <= 128: there one launch beats the GEMM + epilogue pair (c1, d = 64,
  // K = 4, 4096 points: 13.8 vs 15.3 us); at d = 256 (c2, 8192 points) the GEMM's
  // staged P outruns the fused kernel's P stream (28.4 + 7.8 vs 43.9 us)
  const int dp = (m.d + 31) / 32 * 32;
  return a.kind == 0 && !a.zero_mu && m.d >= 1 && dp <= 128 && m.K >= 1 && m.K <= kMaxK &&
         (int64_t)m.K * dp <= 16 * 4 * kMaxSlots && m.P64 && m.mu64 &&
         (m.family == SB_FAMILY_GAUSS_MIX || (m.family == SB_FAMILY_STUDENT_T && m.K == 1));
}

int launch_fused_logl_grad(const Model &m, const ASrc &a, int64_t M, const int32_t *count,
                           const int32_t *outmap, double *logl, double *grad, int64_t ldg,
                           double *aux, hipStream_t s) {
  if (!fused_logl_grad_ok(m, a)) {
    set_error("fused logL+grad: unsupported model or operand");
    return SB_E_UNSUPPORTED;
  }
  if (M <= 0) return SB_OK;
  FusedArgs f;
  f.m = m;
  f.a = a;
  f.M = M;
  f.count = count;
  f.outmap = outmap;
  f.logl = logl;
  f.grad = grad;
  f.ldg = ldg;
  f.aux = aux;
  f.dp = (m.d + 31) / 32 * 32;
  const int nbk = f.dp / 16;
  // one row block of 16 points per workgroup: two (32 points) measured slower
  // at d = 64, K = 4 and d = 256 (one wave per SIMD at 290 registers) and would
  // take more than 64 KB of LDS there
  const size_t lds = fused::lds_bytes(m.K, f.dp);
  const dim3 grid((unsigned)ceil_div(M, fused::kRows));
  const bool fast = m.d % 8 == 0 && (((uintptr_t)m.P64) & 15) == 0;
  switch ((m.K * nbk + 3) / 4) {  // 16-column blocks per wave
    case 1: launch_fused<1>(fast, grid, lds, s, f); break;
    case 2: launch_fused<2>(fast, grid, lds, s, f); break;
    case 3: launch_fused<3>(fast, grid, lds, s, f); break;
    case 4: launch_fused<4>(fast, grid, lds, s, f); break;
    case 5: launch_fused<5>(fast, grid, lds, s, f); break;
    default: launch_fused<6>(fast, grid, lds, s, f); break;
  }
  SB_LAUNCH_CHECK();
  return SB_OK;
}

}  // namespace sb
