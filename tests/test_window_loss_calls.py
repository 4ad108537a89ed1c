"""The window loss under what follows or rewrites torch's operations: a kernel launched on raw pointers
shows nothing to it, so such calls take the composed form."""
import pytest

torch = pytest.importorskip("torch")

from torch.fx.experimental.proxy_tensor import make_fx  # noqa: E402
from torch.overrides import TorchFunctionMode  # noqa: E402
from torch.utils._python_dispatch import TorchDispatchMode  # noqa: E402


class Ops(TorchDispatchMode):
    def __init__(self):
        super().__init__()
        self.names = []

    def __torch_dispatch__(self, func, types, args=(), kwargs=None):
        self.names.append(func.overloadpacket.__name__)
        return func(*args, **(kwargs or {}))


class Calls(TorchFunctionMode):
    def __torch_function__(self, func, types, args=(), kwargs=None):
        return func(*args, **(kwargs or {}))


def test_what_watches_the_operations():
    from paper_2002_00250_amd.adjoint import _watched
    assert not _watched()
    with torch.device("cpu"):                 # a default device only places new tensors
        assert not _watched()
        with Calls():
            assert _watched()
    with Ops():
        assert _watched()
    seen = []

    def f(x):
        seen.append(_watched())
        return x * 2

    for mode in ("real", "fake", "symbolic"):
        for pre in (False, True):
            make_fx(f, tracing_mode=mode, pre_dispatch=pre)(torch.ones(3))
    torch.func.vmap(f)(torch.ones(3))
    torch.func.jvp(f, (torch.ones(3),), (torch.ones(3),))
    assert all(seen) and len(seen) == 8
    assert not _watched()


@pytest.fixture
def case():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    g = torch.Generator(device="cuda").manual_seed(4)
    Z = torch.randn((4, 6, 10), device="cuda", generator=g) * 2
    has = (torch.rand(Z.shape, device="cuda", generator=g) < 0.8).to(torch.uint8)
    gt = (torch.rand(Z.shape, device="cuda", generator=g) < 0.4).to(torch.uint8) * 255
    return Z, has, gt


def _grad(f, Z, *args):
    z = Z.detach().clone().requires_grad_()
    loss = f(z, *args)
    loss.backward()
    return loss.detach(), z.grad


CLOSE = dict(rtol=1e-5, atol=1e-8)


@pytest.mark.gpu
@pytest.mark.parametrize("mode", ["real", "fake"])
def test_a_trace_holds_the_loss(case, mode):
    from paper_2002_00250_amd import adjoint
    Z, has, gt = case
    traced = make_fx(lambda z, h, t: adjoint.window_bce_loss(z, h, t, 1, 0.7), tracing_mode=mode)(Z, has, gt)
    step = make_fx(lambda z, h, t: torch.autograd.grad(adjoint.window_bce_loss(z, h, t, 1, 0.7), z)[0],
                   tracing_mode=mode)(Z.clone().requires_grad_(), has, gt)
    for scale in (1.0, -0.5):
        want, grad = _grad(adjoint._bce_torch, Z * scale, has, gt, 1, 0.7)
        assert torch.allclose(traced(Z * scale, has, gt), want, **CLOSE)
        assert torch.allclose(step((Z * scale).requires_grad_(), has, gt), grad, **CLOSE)


@pytest.mark.gpu
def test_modes_see_the_operations(case):
    from paper_2002_00250_amd import adjoint
    Z, has, gt = case
    want, grad = _grad(adjoint._bce_torch, Z, has, gt, 1, 1.0)
    with Ops() as ops:
        loss, g = _grad(adjoint.window_bce_loss, Z, has, gt)
    assert "binary_cross_entropy_with_logits" in ops.names
    assert torch.allclose(loss, want, **CLOSE) and torch.allclose(g, grad, **CLOSE)
    z = Z.clone().requires_grad_()
    loss = adjoint.window_bce_loss(z, has, gt)    # the loss before the mode, its gradient inside
    with Ops() as ops:
        loss.backward()
    assert len(ops.names) > 3 and torch.allclose(z.grad, grad, **CLOSE)
    with Calls():
        assert torch.allclose(adjoint.window_bce_loss(Z, has, gt), want, **CLOSE)
    with torch.device("cuda"):
        assert adjoint._bce_kernel_takes(Z, has, gt, 1, 1.0)
