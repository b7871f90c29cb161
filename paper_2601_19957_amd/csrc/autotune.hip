// Tile-shape autotuner for the quadratic-form GEMM.
//
// The first time a shape class (dtype, d, K, M rounded up to a power of two)
// is seen, each candidate tile (BM x BN x k-tile: four for FP64, for FP32 and
// for BF16 at d % 8 != 0, seven with their LDS stages for the BF16 and split
// contractions) is timed with HIP events, one warm-up and five timed launches,
// and the fastest is cached for the process.  The launches run on the caller's probe (its operands and
// scratch outputs, which the real launch overwrites).  Timing synchronises the
// stream, so a stream under graph capture gets the heuristic choice (not
// cached).  SB_TILE=BMxBN[xBK[xSTAGES]] forces a shape; SB_AUTOTUNE=0 uses the
// heuristic without timing.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <map>
#include <mutex>
#include <tuple>

#include "internal.h"

namespace sb {

namespace {
std::mutex g_mu;
std::map<std::tuple<int, int, int, int, int, int>, TileCfg> g_cache;

int bucket(int64_t M) {
  int b = 0;
  while ((1ll << b) < M) ++b;
  return b;
}

TileCfg heuristic(int dtype, int d, int64_t M) {
  TileCfg t;  // BF16 kernels: 128 rows, 128 -> a 32-wide k-tile
  t.bn = (d <= 64) ? 64 : 128;
  t.bm = (M <= 4096 || d <= 64) ? 64 : 128;
  if (dtype == DT_F64 || dtype == DT_F32) {
    // FP64, FP32: narrow tiles while rows are few (1000 x 203, K = 3 in FP64:
    // 16.5 us against 24), else 64 x 128 x 16
    t.bm = 64;
    t.bn = (M <= 4096 || d <= 64) ? 64 : 128;
    t.bk = t.bn == 64 ? 32 : 16;
  }
  return t;
}

// Times the candidates of one launch; returns false on any runtime error (the
// caller then uses the heuristic).
bool time_launches(int dtype, const Model &m, const ASrc &a, QuadOut o, int64_t M, hipStream_t s,
                   TileCfg *best) {
  const bool bf = (dtype == DT_BF16 || dtype == DT_F32S) && quad_gemm_bf16_ok(m.d);
  hipEvent_t e0, e1;
  bool ok = hipEventCreate(&e0) == hipSuccess;
  ok = ok && hipEventCreate(&e1) == hipSuccess;
  float best_ms = 0.f;
  bool have = false;
  // (BM, BN, k-tile, stages) of the matrix-core kernels: FP64 and FP32 (32 rows:
  // FP64 only), BF16 where d % 8 != 0 (one k-tile), BF16.  FP64 at 16384 x 1024, K =
  // 8: 128 x 128 x 16 4.19 ms, 64 x 128 x 32 4.31, 64 x 64 x 32 4.34, 64 x 128 x 16
  // 4.41, 128 x 64 x 32 4.42, 32 x 64 x 32 4.90; with K = 1 0.540, 0.550, 0.545, 0.559,
  // 0.564, 0.649; at 1000 x 203, K = 3: 32 x 64 x 32 15.0 us, 64 x 64 x 32 15.9, 64 x
  // 128 x 16 23.1.  FP32 at 16384 x 1024, K = 8: 64 x 128 x 16 2.08 ms, 128 x 128 x 16
  // 2.10, 64 x 128 x 32 2.17, 64 x 64 x 32 2.23; at 8192 x 256: 64 x 64 x 32 16.2 us,
  // 64 x 128 x 32 16.4, 64 x 128 x 16 16.6.
  const int cands_f64[4][4] = {{32, 64, 32, 1}, {64, 64, 32, 1}, {64, 128, 16, 1},
                               {128, 128, 16, 1}};
  const int cands_f32[4][4] = {{64, 64, 32, 1}, {64, 128, 16, 1}, {64, 128, 32, 1},
                               {128, 128, 16, 1}};
  const int cands_b16[4][4] = {{64, 64, 32, 1}, {128, 64, 32, 1}, {64, 128, 32, 1},
                               {128, 128, 32, 1}};
  const int cands_bf[7][4] = {{128, 128, 32, 1}, {128, 128, 64, 1}, {256, 128, 32, 1},
                              {128, 256, 32, 1}, {256, 256, 32, 1}, {128, 128, 32, 2},
                              {256, 256, 32, 2}};
  const int nc = bf ? 7 : 4;
  for (int c = 0; c < nc && ok; ++c) {
    TileCfg t;
    const int *cd = bf                   ? cands_bf[c]
                    : dtype == DT_F64  ? cands_f64[c]
                    : dtype == DT_BF16 ? cands_b16[c]
                                       : cands_f32[c];
    t.bm = cd[0];
    t.bn = cd[1];
    t.bk = cd[2];
    t.stages = cd[3];
    // ray points run only the 32-wide k-tiles, no 256 x 128, and two stages only for
    // the BF16 operand
    if (bf && a.kind == 1 &&
        (t.bk != 32 || (t.stages != 1 && dtype != DT_BF16) || (t.bm == 256 && t.bn == 128)))
      continue;
    ok = launch_quad_gemm(dtype, m, a, M, nullptr, o, t, s) == SB_OK;  // warm-up
    ok = ok && hipEventRecord(e0, s) == hipSuccess;
    for (int r = 0; r < 5 && ok; ++r) ok = launch_quad_gemm(dtype, m, a, M, nullptr, o, t, s) == SB_OK;
    ok = ok && hipEventRecord(e1, s) == hipSuccess;
    ok = ok && hipEventSynchronize(e1) == hipSuccess;
    float ms = 0.f;
    ok = ok && hipEventElapsedTime(&ms, e0, e1) == hipSuccess;
    // FP64, FP32: a later candidate has to be 3% faster.  Near ties are settled
    // by the order and not by the noise of one timing, and the smaller tile
    // comes first, which loses less when fewer rows than these are active.
    if (ok && (!have || ms < (bf ? 1.f : 0.97f) * best_ms)) {
      have = true;
      best_ms = ms;
      *best = t;
    }
  }
  if (ok) ok = hipStreamSynchronize(s) == hipSuccess;
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  (void)hipGetLastError();
  return ok;
}

}  // namespace

bool parse_tile(const char *e, TileCfg *t) {
  int bm = 0, bn = 0, bk = 32, st = 1;
  if (!e || sscanf(e, "%dx%dx%dx%d", &bm, &bn, &bk, &st) < 2) return false;
  t->bm = bm;
  t->bn = bn;
  t->bk = bk;
  t->stages = st;
  return true;
}

TileCfg autotune_tiles(int dtype, const Model &m, int64_t M, hipStream_t s, const TuneProbe *probe) {
  {
    TileCfg t;
    if (parse_tile(getenv("SB_TILE"), &t)) return t;
  }
  const char *at = getenv("SB_AUTOTUNE");
  const bool timed = !(at && at[0] == '0');
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(s, &cs) != hipSuccess) cs = hipStreamCaptureStatusNone;
  auto heur = [&]() { return heuristic(dtype, m.d, M); };
  if (!timed || cs != hipStreamCaptureStatusNone || M <= 0) return heur();
  std::lock_guard<std::mutex> lk(g_mu);
  int dev = 0;
  (void)hipGetDevice(&dev);
  // (the operand kind and the sum-of-squares mode select kernels of their own)
  const int variant = probe ? probe->a.kind + 2 * (probe->o.sumsq ? 1 : 0) : 0;
  auto key = std::make_tuple(dev, dtype, m.d, m.K, bucket(M), variant);
  auto it = g_cache.find(key);
  if (it != g_cache.end()) return it->second;
  TileCfg t = heur();
  if (!probe) return t;  // no buffers to time on: heuristic, not cached
  // a prefix of the caller's launch is enough to rank the tiles
  const bool ok =
      time_launches(dtype, m, probe->a, probe->o, std::min<int64_t>(M, 65536), s, &t);
  if (!ok) t = heur();
  g_cache[key] = t;
  return t;
}

}  // namespace sb
