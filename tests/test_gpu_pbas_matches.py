"""PBAS with a match count of two (kept as the two smallest distances) and of others (counted),
against the oracle bit for bit: few samples with depth, thresholds at and above the byte range,
where an empty depth slot must never pass for a match."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from gpu_util import compare_pbas_grad_state, compare_pbas_state, to_dev  # noqa: E402
from oracle.pbas import PbasParams, PbasRef  # noqa: E402
from test_gpu_parity import _model  # noqa: E402


@pytest.mark.parametrize("R", [18.0, 255.0, 255.5, 300.0])
@pytest.mark.parametrize("N,matches", [(2, 2), (3, 2), (8, 2), (9, 2), (21, 2), (36, 2), (3, 1), (9, 3), (36, 3)])
def test_match_counts(N, matches, R):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2002_00250_amd import fgs
    H, W = 9, 67
    p = PbasParams(N=N, min_matches=matches, R_lower=(R, R, R, R))
    ref, m = PbasRef(H, W, p), _model(fgs.FGS_PBAS, H, W, p)
    rng = np.random.default_rng(N)
    for t in range(N + 14):
        rgb = rng.integers(0, 256, (H, W, 3)).astype(np.uint8)
        depth = np.where(rng.random((H, W)) < 0.15, rng.integers(1, 5000, (H, W)), 0).astype(np.uint16)
        exp = ref.step(rgb, depth)
        m.push(*to_dev(rgb, depth))
        assert np.array_equal(m.mask_host(), exp), t
    res = compare_pbas_state(m.state(), ref.state_planes())
    assert all(v == 0 for v in res.values()), res
    m.close()


@pytest.mark.parametrize("N,matches", [(2, 2), (9, 2), (20, 2), (33, 2), (3, 1), (20, 3), (33, 1)])
def test_match_counts_with_gradients(N, matches):
    """The gradient variant's two ways to count, the same frames and thresholds."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2002_00250_amd import fgs
    H, W = 9, 67
    p = PbasParams(N=N, min_matches=matches, gradient=True, grad_alpha=7.0, R_lower=(60.0, 60.0, 60.0, 300.0))
    ref, m = PbasRef(H, W, p), _model(fgs.FGS_PBAS, H, W, p)
    rng = np.random.default_rng(N)
    for t in range(N + 14):
        rgb = rng.integers(0, 256, (H, W, 3)).astype(np.uint8)
        depth = np.where(rng.random((H, W)) < 0.15, rng.integers(1, 5000, (H, W)), 0).astype(np.uint16)
        exp = ref.step(rgb, depth)
        m.push(*to_dev(rgb, depth))
        assert np.array_equal(m.mask_host(), exp), t
    res = compare_pbas_grad_state(m.state(), ref.state_planes())
    assert all(v == 0 for v in res.values()), res
    m.close()
