"""The window's loss kernels against the composed form in float64: value to 1e-6 of it (each
term a few float32 roundings, 6e-8 each, sums in fp64), gradient to 1e-6 of a full term's
|w g / (sum w tau)|.  And the calls that the kernels leave to the composed form."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2002_00250_amd import fgs
    fgs.lib()
    yield


def _case(T, H, W, seed, spread=6.0):
    g = torch.Generator(device="cuda").manual_seed(seed)
    Z = torch.randn((T, H, W), device="cuda", generator=g) * spread
    has = (torch.rand((T, H, W), device="cuda", generator=g) < 0.8).to(torch.uint8)
    gt = (torch.rand((T, H, W), device="cuda", generator=g) < 0.4).to(torch.uint8) * 255
    return Z, has, gt


@pytest.mark.parametrize("T,H,W", [(1, 1, 1), (2, 1, 1), (5, 7, 9), (3, 64, 64), (9, 33, 47), (4, 512, 517)])
@pytest.mark.parametrize("t0,tau", [(0, 1.0), (1, 1.0), (-1, 0.7), (2, 3)])
def test_loss_and_gradient(T, H, W, t0, tau):
    from paper_2002_00250_amd import adjoint
    t0 = T - 1 if t0 < 0 else t0
    if t0 >= T:
        pytest.skip("no frame left")
    Z, has, gt = _case(T, H, W, T * H + W)
    if W == 9:
        has = has * 3                      # weights need not be 0 or 1
    if W == 47:
        has, gt = torch.zeros_like(has), gt > 0
    if H == 64:
        Z = Z * 1.0e4
    Z.requires_grad_()
    assert adjoint._bce_kernel_takes(Z, has, gt, t0, tau)
    loss = adjoint.window_bce_loss(Z, has, gt, t0, tau)
    (3.0 * loss).backward()
    Z64 = Z.detach().double().requires_grad_()
    want = adjoint._bce_torch(Z64, has, gt, t0, tau)
    (3.0 * want).backward()
    assert abs(loss.item() - want.item()) <= 1e-6 * abs(want.item())
    full = 3.0 * has.double() / max(1.0, has[t0:].double().sum().item()) / tau
    off = (Z.grad.double() - Z64.grad).abs()
    assert bool((off <= 1e-6 * full).all()) and bool((Z.grad[:t0] == 0).all())


def test_values_that_are_not_finite():
    from paper_2002_00250_amd import adjoint
    for bad in (float("inf"), float("-inf"), float("nan")):
        for where in (True, False):        # under a weight, and without one
            Z, has, gt = _case(3, 5, 7, 1)
            Z[2, 3, 4], has[2, 3, 4] = bad, int(where)
            for truth in (0, 255):
                gt[2, 3, 4] = truth
                a, b = Z.clone().requires_grad_(), Z.clone().requires_grad_()
                la, lb = adjoint.window_bce_loss(a, has, gt), adjoint._bce_torch(b, has, gt, 1, 1.0)
                la.backward()
                lb.backward()
                assert np.array_equal(np.isfinite(la.item()), np.isfinite(lb.item()))
                assert np.isnan(la.item()) == np.isnan(lb.item())
                assert torch.allclose(a.grad, b.grad, rtol=1e-5, atol=1e-9, equal_nan=True)


def test_calls_left_to_the_composed_form():
    from paper_2002_00250_amd import adjoint
    f = adjoint.window_bce_loss
    Z, has, gt = _case(4, 6, 10, 2, spread=1.5)
    ref = adjoint._bce_torch
    close = dict(rtol=1e-5, atol=1e-8)
    # a strided score tensor, other types, the CPU, an empty range
    S = torch.randn((4, 6, 20), device="cuda")[..., ::2]
    assert torch.allclose(f(S, has, gt), ref(S, has, gt, 1, 1.0), **close)
    assert torch.allclose(f(Z.double(), has, gt), ref(Z.double(), has, gt, 1, 1.0), **close)
    assert torch.allclose(f(Z.cpu(), has.cpu(), gt.cpu()), ref(Z, has, gt, 1, 1.0).cpu(), **close)
    assert f(Z, has, gt, t0=4).item() == 0.0
    # a batch of scores, forward-mode differentiation
    B = torch.stack([Z, 2 * Z])
    got = torch.func.vmap(lambda z: f(z, has, gt))(B)
    assert torch.allclose(got, torch.stack([ref(b, has, gt, 1, 1.0) for b in B]), **close)
    d = torch.randn_like(Z)
    _, t = torch.func.jvp(lambda z: f(z, has, gt), (Z,), (d,))
    _, u = torch.func.jvp(lambda z: ref(z, has, gt, 1, 1.0), (Z,), (d,))
    assert torch.allclose(t, u, **close)
    # the gradient differentiated, and batched
    out = []
    for g in (f, lambda *a: ref(*a, 1, 1.0)):
        z = Z.clone().requires_grad_()
        (first,) = torch.autograd.grad(g(z, has, gt), z, create_graph=True)
        (second,) = torch.autograd.grad((first * d).sum(), z)
        z = Z.clone().requires_grad_()
        (batch,) = torch.autograd.grad(g(z, has, gt), z, torch.tensor([1.0, 2.0, -3.0], device="cuda"),
                                       is_grads_batched=True)
        out.append((first.detach(), second, batch))
    for a, b in zip(*out):
        assert torch.allclose(a, b, **close)
    # saved-tensor hooks see what is kept
    seen = []
    with torch.autograd.graph.saved_tensors_hooks(lambda x: (seen.append(x.shape), x.clone())[1], lambda x: x):
        z = Z.clone().requires_grad_()
        f(z, has, gt).backward()
    assert Z.shape in seen and torch.allclose(z.grad, out[0][0], **close)


def test_replays_in_a_captured_graph():
    from paper_2002_00250_amd import adjoint
    Z, has, gt = _case(3, 40, 50, 3)
    Z.requires_grad_()
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        adjoint.window_bce_loss(Z, has, gt).backward()
    torch.cuda.current_stream().wait_stream(s)
    Z.grad = None
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        loss = adjoint.window_bce_loss(Z, has, gt)
        (grad,) = torch.autograd.grad(loss, Z)
    for k in range(3):
        with torch.no_grad():
            Z.mul_(0.5 + k)
        graph.replay()
        torch.cuda.synchronize()
        z = Z.detach().clone().requires_grad_()
        want = adjoint._bce_torch(z, has, gt, 1, 1.0)
        want.backward()
        assert torch.allclose(loss, want, rtol=1e-5) and torch.allclose(grad, z.grad, rtol=1e-4, atol=1e-9)
