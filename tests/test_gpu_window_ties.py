"""The window's ranking near ties of the rank keys: it sorts by approximate keys where adjacent ranks are
clearly apart, and again by the rounded ones, equal keys by their rank before, where the sorted ones are
not.  Three unmatched values A, C, B in turn leave the ranks (A, C, B) with A and B at one key where the
replacement weight is (sqrt(5) - 1) / 2 of the decay: C is out of order, and A and B meet only by the sort.
The replacement weight is swept over float32 steps about that, and records and scores are the oracle's."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from oracle.adjoint import record_window  # noqa: E402
from oracle.gmm import GmmParams  # noqa: E402
from test_gpu_adjoint import _decode, _dev, _params_c  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2002_00250_amd import fgs
    fgs.lib()
    yield


def _frames(rng, H, W):
    """A, C, B and three more of them at random, far apart in every channel and in depth."""
    order = [0, 2, 1] + list(rng.integers(0, 3, 3))
    level = np.stack([rng.integers(0, 30, (H, W, 3)) + 90 * k for k in range(3)])
    depth = np.stack([rng.integers(0, 300, (H, W)) + 500 + 3000 * k for k in range(3)])
    return level[order].astype(np.uint8), depth[order].astype(np.uint16)


def _check(K, H, W, alpha, step, seen):
    from paper_2002_00250_amd.adjoint import GmmWindow
    a = 1.0 - np.float32(alpha)
    w = np.float32(a * (np.sqrt(5.0) - 1.0) / 2.0)
    w = (w.view(np.int32) + np.int32(step)).view(np.float32)
    p = GmmParams(Kc=K, Kd=K, alpha=alpha, w_init=float(w))
    small = min(H, 8), min(W, 8)
    rgb, dep = _frames(np.random.default_rng(step + 100), *small)
    reps = -(-H // small[0]), -(-W // small[1])
    big = [np.tile(x, (1, *reps) + (1,) * (x.ndim - 3))[:, :H, :W] for x in (rgb, dep)]
    T = rgb.shape[0]
    with np.errstate(divide="ignore", invalid="ignore"):
        Z, has, dc, dd = record_window(rgb, dep, p)
    win = GmmWindow(T, H, W, _params_c(p), checkpoint_every=T)
    Zg, hg = win.forward(torch.tensor([p.alpha, p.lam, p.w_depth], device="cuda"), *_dev(*big))
    rec = win.records()
    win.close()

    def whole(x):
        return np.tile(x, (1,) * (x.ndim - 2) + reps)[..., :H, :W]

    assert np.array_equal(Zg.cpu().numpy(), whole(Z)) and np.array_equal(hg.cpu().numpy() != 0, whole(has))
    for dec, shift in ((dc, 0), (dd, 32)):
        term, argmin, active, ks, clamp, perm = _decode(rec, K, shift)
        assert np.array_equal(perm, whole(dec.perm)) and np.array_equal(ks, whole(dec.kstar))
        assert np.array_equal(np.where(term, argmin, 0), whole(np.where(dec.term, dec.argmin, 0)))
        seen.update(tuple(v) for v in dec.perm[2].reshape(K, -1).T)


@pytest.mark.parametrize("K", [3, 4, 5])
@pytest.mark.parametrize("alpha", [0.01, 0.125])
def test_near_ties(K, alpha):
    seen = set()
    for step in range(-20, 21):               # a small window: the mixtures on wavefronts of their own
        _check(K, 8, 8, alpha, step, seen)
    for step in (-3, -1, 0, 1, 3):            # a large one
        _check(K, 364, 363, alpha, step, seen)
    # A first (or equal, and first before) and B first
    assert {s[:2] for s in seen} == {(0, K - 1), (K - 1, 0)}, seen
