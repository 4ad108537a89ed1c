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


@pytest.mark.gpu
@pytest.mark.parametrize("t0", [0, 1, 3])
def test_the_caller_may_refill_what_it_passed(case, t0):
    """Scores, flags and truth are the caller's again after the loss, as with the composed form, which
    keeps converted copies: the gradient is that of the values the loss was taken of."""
    from paper_2002_00250_amd import adjoint, fgs
    Z, has, gt = case
    has = has * 3
    want, grad = _grad(adjoint._bce_torch, Z, has, gt, t0, 0.7)
    T, H, W = Z.shape
    m = fgs.Model(fgs.FGS_GMM, H, W)
    for v in (0, 200):
        m.push(torch.full((H, W, 3), v, dtype=torch.uint8, device="cuda"),
               torch.full((H, W), 900, dtype=torch.int16, device="cuda"))
    z = Z.clone().requires_grad_()
    s, h, t = z * 1.0, has.clone(), gt.clone()
    assert adjoint._bce_kernel_takes(s, h, t, t0, 0.7)
    loss = adjoint.window_bce_loss(s, h, t, t0, 0.7)
    m.mask_into(t[T - 1])                     # (the library's writes show on no version counter)
    m.mask_into(h[T - 1])
    t[:T - 1] = 255 - t[:T - 1]
    h.fill_(1)
    s.detach().mul_(-2.0)
    with torch.no_grad():
        s.add_(1.0)
    loss.backward()
    assert torch.allclose(loss, want, **CLOSE) and torch.allclose(z.grad, grad, **CLOSE)
    m.close()


@pytest.mark.gpu
@pytest.mark.parametrize("t0,weight", [(0, 1), (1, 3), (2, 255)])
def test_gradients_of_gradients(case, t0, weight):
    from paper_2002_00250_amd import adjoint
    Z, has, gt = case
    has = has * weight
    out = []
    for f in (adjoint.window_bce_loss, adjoint._bce_torch):
        z, c = Z.clone().requires_grad_(), torch.tensor(1.5, device="cuda", requires_grad=True)
        loss = c * f(z, has, gt, t0, 0.7)
        (first,) = torch.autograd.grad(loss, z, create_graph=True)
        second = torch.autograd.grad((first ** 2).sum(), (z, c), create_graph=True)
        (third,) = torch.autograd.grad(second[0].sum(), z)
        out.append((loss, first, *second, third))
    for a, b in zip(*out):
        scale = float(b.detach().abs().max())
        assert torch.allclose(a, b, rtol=1e-4, atol=1e-5 * scale)


@pytest.mark.gpu
def test_hooks_that_give_back_something_else(case):
    """Saved-tensor hooks that hand the backward other tensors than they were given."""
    from paper_2002_00250_amd import adjoint
    Z, has, gt = case
    want, grad = _grad(adjoint._bce_torch, Z, has, gt, 1, 1.0)
    wide = lambda x: torch.stack([x, x], -1)[..., 0]  # noqa: E731
    for unpack in (lambda x: x, wide, lambda x: x.float() if x.is_floating_point() else x):
        with torch.autograd.graph.saved_tensors_hooks(lambda x: x.clone(), unpack):
            loss, g = _grad(adjoint.window_bce_loss, Z, has, gt)
        assert torch.allclose(loss, want, **CLOSE) and torch.allclose(g, grad, **CLOSE)


@pytest.mark.gpu
@pytest.mark.parametrize("T,H,W", [(1, 1, 1), (3, 1, 1), (3, 1, 2), (5, 7, 9), (3, 64, 64), (2, 333, 1001)])
@pytest.mark.parametrize("shift", [0, 1])
def test_with_and_without_a_gradient(T, H, W, shift):
    """The same loss to the bit, whether the slopes are kept or not; slopes and weights in place."""
    from paper_2002_00250_amd import adjoint
    g = torch.Generator(device="cuda").manual_seed(T * H + W)
    n = T * H * W
    Z = (torch.randn(n + shift, device="cuda", generator=g) * 4)[shift:].view(T, H, W)
    has = (torch.rand((T, H, W), device="cuda", generator=g) < 0.7).to(torch.uint8) * 2
    gt = torch.rand((T, H, W), device="cuda", generator=g) < 0.5
    for t0 in range(min(T, 3)):
        a = adjoint.window_bce_loss(Z, has, gt, t0)
        b = adjoint.window_bce_loss(Z.clone().requires_grad_(), has, gt, t0)
        _, slope, weight, work, i0 = adjoint._bce_forward(Z, has, gt, t0, 1.0, True)
        assert i0 == t0 * H * W
        if shift == 0:
            assert torch.equal(a, b)
        assert torch.equal(weight[t0:], has[t0:]) and not weight[:t0].any() and not slope[:t0].any()
        want = (torch.sigmoid(Z.double()) - gt.double()) * has
        # (a sigmoid of a few roundings and one subtraction, times a weight of 2)
        assert bool(((slope - want).abs()[t0:] <= 5e-7).all())
        assert work[1].item() == max(1.0, has[t0:].double().sum().item())


@pytest.mark.gpu
@pytest.mark.parametrize("reentrant", [False, True])
def test_recomputed_by_a_checkpoint(case, reentrant):
    from paper_2002_00250_amd import adjoint
    from torch.utils.checkpoint import checkpoint
    Z, has, gt = case
    want, grad = _grad(adjoint._bce_torch, Z, has, gt, 1, 1.0)
    for f in (lambda z: adjoint.window_bce_loss(z, has, gt), lambda z: adjoint.window_bce_loss(z * 2, has, gt, 1, 2.0)):
        loss, g = _grad(lambda z: checkpoint(f, z, use_reentrant=reentrant), Z)
        assert torch.allclose(loss, want, **CLOSE) and torch.allclose(g, grad, **CLOSE)


@pytest.mark.gpu
def test_a_graph_kept_for_more_gradients(case):
    from paper_2002_00250_amd import adjoint
    Z, has, gt = case
    _, grad = _grad(adjoint._bce_torch, Z, has, gt, 1, 1.0)
    z = Z.clone().requires_grad_()
    loss = adjoint.window_bce_loss(z, has, gt)
    for k in range(3):
        (g,) = torch.autograd.grad(loss * (k + 1), z, retain_graph=True)
        assert torch.allclose(g, grad * (k + 1), **CLOSE)
    (loss + 2 * adjoint.window_bce_loss(z, has, gt)).backward()
    assert torch.allclose(z.grad, 3 * grad, **CLOSE)
