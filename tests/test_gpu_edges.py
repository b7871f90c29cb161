"""GPU: calls at the far ends of what the entry points take."""
import ctypes as C

import numpy as np
import pytest

import oracle as O
from paper_2601_19957_amd import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def L():
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    from paper_2601_19957_amd import _lib
    return _lib


def dev(a):
    return torch.as_tensor(np.ascontiguousarray(a), device="cuda")


def test_contraction_past_one_launch(L, monkeypatch):
    """FP64 ray points in more tiles than one launch holds (2^24 workgroups of 256 threads):
    33.6 million points x 16 components in 32-row tiles.  The best l of rays at the start, around
    the last row of the first launch and at the end is the oracle's at the sampled points."""
    monkeypatch.setenv("SB_TILE", "32x64x32")
    d, K, R, npts = 5, 16, 32769 + 8, 1024
    assert -(-R * npts // 32) * K > 1 << 24
    rng = np.random.Generator(np.random.PCG64(77))
    prob = synth.gaussian_mixture(rng, d, K, -40.0, 40.0, 0.2, 1.0, 0.0, box_half=45.0)
    out = L.sb_discover_dev(L.DeviceModel(prob), R, npts, 1, 9)
    edge = ((1 << 24) - 1) // K * 32 // npts  # the ray that the first launch's last row is on
    bl = out["ray_best_l"].cpu().numpy()
    t = ((np.arange(npts) + 0.5) / npts)[:, None]
    for r in (0, 1, edge - 1, edge, edge + 1, R - 1):
        p0, p1 = out["P0"][r].cpu().numpy(), out["P1"][r].cpu().numpy()
        want = np.max(O.logl(prob, p0 + t * (p1 - p0), grad=False))
        assert abs(bl[r] - want) <= 1e-11 * max(1.0, abs(want)), r


@pytest.mark.parametrize("R", [1, 5, 64, 65, 130, 512, 513, 1000, 1024, 1040, 3001])
def test_ray_ranking_by_size(L, R):
    """Shares of single keys (up to 512 rays) and of whole 64s (the last of them part empty, and
    waves without any), with many equal maxima: the start rays are those of a stable sort of
    the rays' best l, descending, ties to the lower index."""
    d, npts = 4, 8
    prob = synth.Problem(family=synth.FAMILY_GAUSS_MIX, norm=synth.NORM_DENSITY, d=d, K=1,
                         log_w=np.zeros(1), mu=np.zeros((1, d)),
                         prec=(1e-15 * np.eye(d))[None], nu=0.0, logl_offset=0.0,
                         lo=-np.ones(d), hi=np.ones(d), sum_log_lambda=np.array([d * 34.5]))
    out = L.sb_discover_dev(L.DeviceModel(prob), R, npts, R, 5)
    bl = out["ray_best_l"].cpu().numpy()
    assert R < 64 or len(np.unique(bl)) < R // 2
    assert np.array_equal(out["start_ray"].cpu().numpy(), np.argsort(-bl, kind="stable"))


@pytest.mark.parametrize("d,m,steps", [(129, 8, 20), (203, 8, 20), (203, 12, 24), (255, 8, 20),
                                       (402, 12, 24), (509, 8, 20), (1021, 8, 20), (1022, 12, 24),
                                       (257, 20, 32), (331, 16, 28), (511, 13, 24), (514, 32, 40),
                                       (1023, 32, 40), (67, 16, 28), (129, 20, 32), (255, 32, 40),
                                       (1102, 16, 28)])
def test_lbfgs_path_of_ragged_rows(L, d, m, steps):
    """L-BFGS on rows that end inside a thread's chunk, one wave and several, history in
    registers and streamed: the FP64 points after `steps` accepted steps are the oracle's (whose own
    paths move by at most 1.5e-14 relative under 1e-15 perturbations of these starts; 1e-10 leaves
    room for d-term sums in another order at each step).  In FP32 and with the BF16 history the
    iterations to |grad| <= 2e-4 stay within 1.5 and 2 times the oracle's 40 to 48 (steepest descent
    at this condition number, 50, needs about 290)."""
    rng = np.random.Generator(np.random.PCG64(760 + d))
    P, _ = synth.random_precision(rng, d, 0.02, 1.0)
    mu = rng.uniform(-2, 2, (1, d))
    prob = synth.Problem(0, 0, d, 1, np.zeros(1), mu, P[None], 0.0, 0.0, -9 * np.ones(d),
                         9 * np.ones(d), np.zeros(1))
    X0 = mu + rng.uniform(-3, 3, (4, d))
    md = L.DeviceModel(prob, low_precision=True)
    out = L.sb_lbfgs_dev(md, dev(X0), m=m, max_iter=steps, grad_tol=1e-14)
    x = out["x"].cpu().numpy()
    op = O.OracleProblem(prob)
    for s in range(4):
        r = O.lbfgs(prob, X0[s], m=m, max_iter=steps, grad_tol=1e-14, op=op)
        assert np.max(np.abs(x[s] - r["x"])) <= 1e-10 * max(1.0, np.max(np.abs(r["x"]))), s
    want = max(O.lbfgs(prob, x0, m=m, max_iter=400, grad_tol=2e-4, op=op)["iters"] for x0 in X0)
    for h16 in (False, True) if m == 8 else (False,):
        it = L.sb_lbfgs_dev(md, dev(X0).float(), m=m, grad_tol=2e-4, max_iter=400,
                            hist_bf16=h16)["iters"]
        assert int(it.max()) <= (2.0 if h16 else 1.5) * want


@pytest.mark.parametrize("n,C", [(65, 300), (129, 100), (200, 60), (320, 33), (450, 12), (1024, 4)])
def test_cholesky_batch_equals_single(L, n, C):
    """Batches whose first panels have more tiles than the chip has CUs (their rows solved by a
    launch of their own, the last panels' not) against the same matrices one at a time: the
    same bits, with matrices among them whose pivot fails in the first, a middle and the last
    column (info is that column in both)."""
    A = np.repeat(synth.random_spd(n, 70 + n, cond=1e3, batch=4), -(-C // 4), axis=0)[:C].copy()
    A *= np.linspace(1.0, 3.0, C)[:, None, None]
    fails = {1: 0, 2: n // 2, 3: n - 1}
    for c, k in fails.items():
        A[c, k, k] = -1.0
    Lb, ld, info = L.sb_cholesky_logdet_dev(dev(A))
    assert [int(info[c]) for c in fails] == [k + 1 for k in fails.values()]
    for c in list(range(min(C, 5))) + [C // 2, C - 1]:
        L1, ld1, info1 = L.sb_cholesky_logdet_dev(dev(A[c:c + 1]))
        assert int(info1[0]) == int(info[c])
        if c not in fails:
            assert int(info[c]) == 0
            assert torch.equal(Lb[c], L1[0]) and torch.equal(ld[c], ld1[0])


SIZE_SRC = "__device__ double size(const double *x, int d, const double *p) { return blockDim.x; }"
SUM_SRC = r"""
__device__ double wsum(const double *x, int d, const double *p) {
  double s = 0.0;
  for (int i = 0; i < d; ++i) s += p[i] * x[i];
  return s;
}
"""


@pytest.mark.parametrize("d,n,staged", [(2, 4096, False), (8, 1 << 20, True), (12, 1 << 20, False),
                                        (64, 65536, True), (64, 65600, False),
                                        (64, 393216, True), (96, 49152, True),
                                        (96, 49216, False), (128, 64, False), (512, 4096, False),
                                        (1022, 64, False)])
def test_user_points_staged_where_it_gains(L, d, n, staged):
    """Which kernel takes l at given points (the workgroup's size tells: 64 staged, 256 direct)
    on both sides of the rule's lines, and the values there: a weighted sum within d roundings."""
    X = torch.rand((n, d), dtype=torch.float64, device="cuda") - 0.5
    assert float(L.UserLogL(SIZE_SRC, "size").logl(X[:1].expand(n, d).contiguous())[n - 1]) == (
        64.0 if staged else 256.0)
    p = torch.rand(d, dtype=torch.float64, device="cuda") + 0.5
    l = L.UserLogL(SUM_SRC, "wsum").logl(X, p)
    assert float((l - X @ p).abs().max()) <= 2 * d * 2.0 ** -52 * d


@pytest.mark.parametrize("d,B,staged", [(78, 600, True), (96, 251, True), (96, 256, False),
                                        (96, 2100, True), (160, 76, True), (160, 77, False),
                                        (510, 4, True), (510, 5, False), (2046, 1, False)])
def test_user_differences_staged_where_it_gains(L, d, B, staged):
    """The same for the rows of finite differences, formed in LDS or in memory, and the
    gradient of a weighted sum on either side: its differences round d times each."""
    X = torch.rand((B, d), dtype=torch.float64, device="cuda") - 0.5
    l = L.UserLogL(SIZE_SRC, "size").fd(X, 1e-3)["l"]
    assert float(l[B - 1]) == (64.0 if staged else 256.0)
    p = torch.rand(d, dtype=torch.float64, device="cuda") + 0.5
    out = L.UserLogL(SUM_SRC, "wsum").fd(X, 1e-3, p)
    tol = 2 * d * 2.0 ** -52 * d
    assert float((out["l"] - X @ p).abs().max()) <= tol
    assert float((out["grad"] - p).abs().max()) <= 2 * tol / 1e-3


@pytest.mark.parametrize("d", [165, 166])
def test_result_readback_sizes(L, d):
    """Three modes of d = 165 fill the small readback buffer (4096 bytes) exactly, of d = 166 they
    go to the caller's arrays: the same numbers through a context, without one and, where
    only some arrays are wanted, in those; the modes are the oracle's."""
    rng = np.random.Generator(np.random.PCG64(9))
    prob = synth.gaussian_mixture(rng, d, 3, -8.0, 8.0, 0.1, 1.0, 0.0, box_half=12.0)
    cfg = synth.RunConfig(n_rays=256, n_points=32, n_starts=256, seed=3, precision=0)
    ex = L.ExecContext()
    a, b = L.EvidenceRunner(prob, cfg).run(), L.EvidenceRunner(prob, cfg, exec=ex).run()
    ex.close()
    ref = O.reference_modes(prob)
    assert a.n_modes == b.n_modes == ref.n_modes == 3
    assert a.log_z == b.log_z
    for k in ("modes", "mode_log_z", "mode_logl", "log_det_h"):
        assert np.array_equal(getattr(a, k), getattr(b, k)), k
    r, arrs = L._new_result(cfg.max_modes, d)
    r.modes = r.log_det_h = None
    run = L.EvidenceRunner(prob, cfg)
    assert L.lib().sb_evidence_dev(C.byref(run.ll), C.byref(run.box), C.byref(run.c), C.byref(r),
                                   run.ws.data_ptr(), run.ws.numel(), 0) == 0
    assert r.log_z == a.log_z and np.array_equal(arrs[2][:3], a.mode_logl)
    assert not arrs[0].any() and not arrs[3].any()
    want = ref.modes[:3][np.lexsort(ref.modes[:3].T[::-1])]
    got = a.modes[np.lexsort(a.modes.T[::-1])]
    assert np.max(np.abs(got - want)) <= 1e-8


ONE_LAUNCH = [(1, 1, 1, 0), (4, 2, 15, 0), (31, 12, 17, 0), (33, 3, 16, 0), (64, 6, 130, 0),
              (64, 4, 4096, 0), (65, 3, 9, 0), (96, 4, 100, 0), (128, 3, 2048, 0),
              (64, 4, 100, 3), (100, 3, 33, 5)]


@pytest.mark.parametrize("d,K,B,cut", ONE_LAUNCH)
def test_one_launch_is_the_step_launches(L, d, K, B, cut, monkeypatch):
    """The bulk in one launch against step, compaction and evaluation launches of the same
    kernels' arithmetic: evaluations, iterations, the states of the starts and every number of the result
    are the same, also where the iterations are cut short, and with starts that fill no workgroup.
    A context tells which ran: one block graph for up to 256 steps, or one for eight."""
    rng = np.random.Generator(np.random.PCG64(1700 + d))
    span = 30.0 if K > 1 else 8.0
    prob = synth.gaussian_mixture(rng, d, K, -span, span, 0.05, 1.0, 0.0, box_half=1.5 * span)
    cfg = synth.RunConfig(n_rays=max(B, K), n_points=32, n_starts=B, seed=5, precision=0)
    if cut:
        cfg.max_iter = cut

    def run():
        ex, stream = L.ExecContext(), torch.cuda.Stream()
        with torch.cuda.stream(stream):
            r = L.EvidenceRunner(prob, cfg, exec=ex).run(stream)
        n = ex.stats()["launched"]
        ex.close()
        return r, n

    a, na = run()
    monkeypatch.setenv("SB_ONE_LAUNCH", "0")
    b, nb = run()
    assert na == -(-a.iterations // 256) and nb == b.iterations // 8
    assert a.status == b.status
    for k in ("n_modes", "n_grad_evals", "n_logl_evals", "n_hess_evals", "iterations",
              "n_dead_starts", "n_candidates", "n_reps_pre", "n_rejected_nonpd"):
        assert getattr(a, k) == getattr(b, k), k
    if a.status == 0:
        assert a.log_z == b.log_z
    for k in ("modes", "mode_log_z", "mode_logl", "log_det_h"):
        assert np.array_equal(getattr(a, k), getattr(b, k)), k


@pytest.mark.parametrize("C,d,n", [(256, 64, 8), (256, 64, 9), (256, 64, 256), (192, 64, 60),
                                   (193, 64, 60), (1024, 16, 100), (1024, 17, 3), (4096, 3, 40),
                                   (4097, 3, 9), (8192, 1, 20), (8192, 2, 300), (3000, 5, 50),
                                   (496, 33, 496), (100, 100, 100), (16, 1024, 16)])
def test_dedup_many_representatives(L, C, d, n):
    """n clusters, few and all candidates apart, at each number of values a lane takes and on
    both sides of the one-workgroup limits: the oracle's partition exactly, and with room for
    one less the capacity status."""
    rng = np.random.Generator(np.random.PCG64(40 + C + d + n))
    centres = 3.0 * rng.permutation(n)[:, None] * np.ones((1, d)) + rng.uniform(0, 1, (n, d))
    at = np.concatenate([np.arange(n), rng.integers(n, size=C - n)])
    X = centres[at] + 0.1 * rng.uniform(-1, 1, (C, d))
    l = np.round(rng.standard_normal(C), 1)
    ro, rs = O.dedup(X, l, 0.5)
    assert len(rs) == n
    rep_of, reps = L.sb_dedup_dev(dev(X), dev(l), 0.5, max_reps=n)
    assert np.array_equal(rep_of.cpu().numpy(), ro)
    assert np.array_equal(reps.cpu().numpy(), rs)
    if n > 1:
        with pytest.raises(L.SbError) as e:
            L.sb_dedup_dev(dev(X), dev(l), 0.5, max_reps=n - 1)
        assert e.value.status == L.E_CAPACITY


def test_result_of_one_mode_too_many(L):
    """Four modes with room for three: the capacity status, the number found, and the caller's
    arrays as they were."""
    rng = np.random.Generator(np.random.PCG64(12))
    prob = synth.gaussian_mixture(rng, 6, 4, -30.0, 30.0, 0.1, 1.0, 0.0, box_half=40.0)
    cfg = synth.RunConfig(n_rays=512, n_points=32, n_starts=512, seed=3, precision=0)
    full = L.EvidenceRunner(prob, cfg, exec=True).run()
    assert full.status == 0 and full.n_modes == 4
    cfg.max_modes = 3
    r, arrs = L._new_result(3, 6)
    run = L.EvidenceRunner(prob, cfg)
    st = L.lib().sb_evidence_dev(C.byref(run.ll), C.byref(run.box), C.byref(run.c), C.byref(r),
                                 run.ws.data_ptr(), run.ws.numel(), 0)
    assert st == L.E_CAPACITY and r.n_modes == 4 and np.isnan(r.log_z)
    assert not any(a.any() for a in arrs)
