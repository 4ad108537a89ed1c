"""The adjoint's two memory plans: every frame's changed Gaussians kept by the forward, or
checkpoints and a replay per segment (chosen by their sizes).  Both must give the same scores
and, step for step the same operations, the same gradient bit for bit; the gradient must be
the fp64 reference's (1e-5 relative: sums over some 10^4 float32 terms of 6e-8 each)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from gpu_util import log  # noqa: E402
from oracle.gmm import GmmParams  # noqa: E402
from synth import Scene, preset  # noqa: E402
from test_gpu_adjoint import _dev, _oracle_grad, _params_c  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2002_00250_amd import fgs
    fgs.lib()
    yield


@pytest.mark.parametrize("K", [1, 2, 3, 4, 5])
@pytest.mark.parametrize("H,W,alpha", [(17, 29, 0.01), (16, 16, 0.2)])
def test_both_plans_give_the_same_gradient(K, H, W, alpha):
    from paper_2002_00250_amd.adjoint import GmmWindow
    p = GmmParams(Kc=K, Kd=K, alpha=alpha)
    T = 90
    rgb, dep, gt = Scene(preset("adjoint_640x480", H=H, W=W)).frames(0, T)
    theta0 = (alpha, 2.5, 1.0)
    _, dZ, g_ref, _ = _oracle_grad(rgb, dep, gt, p, theta0)
    r, d = _dev(rgb, dep)
    g = torch.from_numpy(dZ.astype(np.float32)).cuda()
    theta = torch.tensor(theta0, dtype=torch.float32, device="cuda")
    out = []
    # 24 T + 24 K bytes against (T / E + E) 24 K: E = 90 keeps every frame for every K, E = 9
    # replays for K <= 4 (19 K < 90 * 4/5)
    for E in (9, 90, 1):
        win = GmmWindow(T, H, W, _params_c(p), checkpoint_every=E)
        Z, has = win.forward(theta, r, d)
        grad = win.backward(theta, r, d, g)
        again = win.backward(theta, r, d, g)   # the forward's buffers are not consumed
        out.append((Z.cpu().numpy(), has.cpu().numpy(), win.records(), grad.cpu().numpy()))
        assert np.array_equal(grad.cpu().numpy(), again.cpu().numpy())
        win.close()
    for o in out[1:]:
        for a, b in zip(out[0], o):
            assert np.array_equal(a, b)
    rel = np.abs(out[0][3] - g_ref) / np.abs(g_ref)
    log(f"K={K} {H}x{W} alpha={alpha}: gradient {out[0][3]} rel to fp64 {rel}")
    assert np.all(rel <= 1e-5)


@pytest.mark.parametrize("K,E", [(3, 4), (3, 1), (5, 4), (2, 4)])
def test_large_window_equals_its_parts(K, E):
    """A window beyond 2^17 pixels (both mixtures on one wavefront) against its two halves (a
    wavefront each from K = 3 on), whose pixels do not meet: the same scores and records, and
    gradients that add up (the sums are fp64 in another order: 1e-12)."""
    from paper_2002_00250_amd.adjoint import GmmWindow
    T, H, W = 5, 364, 363
    assert H * W > 1 << 17 >= H // 2 * W
    g = torch.Generator(device="cuda").manual_seed(K)
    base = torch.randint(0, 256, (H, W, 3), device="cuda", generator=g)
    rgb = (base + torch.randint(-40, 41, (T, H, W, 3), device="cuda", generator=g)).clamp(0, 255).to(torch.uint8)
    dep = torch.randint(-400, 4000, (T, H, W), device="cuda", generator=g).clamp(min=0).to(torch.int16)
    dZ = torch.randn((T, H, W), device="cuda", generator=g)
    theta = torch.tensor([0.05, 2.5, 1.0], device="cuda")
    p = _params_c(GmmParams(Kc=K, Kd=K))
    whole = GmmWindow(T, H, W, p, checkpoint_every=E)
    Z, has = whole.forward(theta, rgb, dep)
    grad, rec, total = whole.backward(theta, rgb, dep, dZ).cpu(), whole.records(), torch.zeros(3, dtype=torch.float64)
    for rows in (slice(0, H // 2), slice(H // 2, H)):
        part = GmmWindow(T, H // 2, W, p, checkpoint_every=E)
        r, d, z = (x[:, rows].contiguous() for x in (rgb, dep, dZ))
        Zp, hp = part.forward(theta, r, d)
        assert torch.equal(Zp.view(torch.int32), Z[:, rows].contiguous().view(torch.int32))
        assert torch.equal(hp, has[:, rows]) and np.array_equal(part.records(), rec[:, rows])
        total += part.backward(theta, r, d, z).cpu()
        part.close()
    # (fp64 sums of n terms of either sign and of order |dZ| x 10^3 at most: n eps times their size)
    assert torch.all((total - grad).abs() <= 1e-12 * (grad.abs() + 1e3 * float(dZ.abs().sum()))), (total, grad)
    whole.close()
