"""GPU: calls at the far ends of what the entry points take."""
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
