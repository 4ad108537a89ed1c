"""The gradient variant's register classes at both ends of each, with the samples cached and
streamed, on images whose sides leave partial tiles and whose rows are strided: masks and
integer state equal to the oracle's, float state bit for bit."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from gpu_util import compare_pbas_grad_state, log, to_dev  # noqa: E402
from oracle.pbas import PbasParams, PbasRef  # noqa: E402
from synth import Scene, preset  # noqa: E402
from test_gpu_pbas_gradient import _pbas_params_c  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2002_00250_amd import fgs
    fgs.lib()
    yield


@pytest.mark.parametrize("N", [2, 8, 9, 16, 17, 20, 21, 24, 25, 32, 33, 40, 41, 64])
@pytest.mark.parametrize("H,W,stream,pad", [(13, 66, 0, 0), (6, 129, 1, 3), (9, 2, 1, 1)])
def test_classes(N, H, W, stream, pad):
    from paper_2002_00250_amd import fgs
    p = PbasParams(N=N, gradient=True, seed=0x77 + N, T_upper=8.0)
    sc = Scene(preset("pbas_640x480", H=H, W=W))
    ref = PbasRef(H, W, p)
    m = fgs.Model(fgs.FGS_PBAS, H, W, _pbas_params_c(p))
    fgs.fgs_set_cache_policy(m.handle, fgs.FGS_CACHE_STREAM if stream else fgs.FGS_CACHE_KEEP)
    diff = 0
    for t in range(N + 14):
        rgb, D, _ = sc.frame(t)
        exp = ref.step(rgb, D)
        r, d = to_dev(np.pad(rgb, ((0, 0), (0, pad), (0, 0))), np.pad(D, ((0, 0), (0, pad))))
        m.push(r[:, :W], d[:, :W])
        diff += int((m.mask_host() != exp).sum())
    res = compare_pbas_grad_state(m.state(), ref.state_planes())
    m.close()
    log(f"pbas gradient class N={N} {H}x{W} stream {stream}: mask diff {diff}, state {res}")
    assert diff == 0 and all(v == 0 for v in res.values())
