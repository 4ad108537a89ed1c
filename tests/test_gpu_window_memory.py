"""A window's device memory: checkpoint_every bounds it (a record of 8 bytes a pixel and frame, a state of
24 K bytes a pixel per checkpoint and per frame of a segment), and within the bound the backward's segments
are chosen.  Whatever they are, scores and gradients are the same to the bit, also for a backward that
follows another one, or is replayed in a captured graph without its forward."""
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


def _params(K):
    from paper_2002_00250_amd import fgs
    p = fgs.fgs_gmm_params_default()
    p.Kc = p.Kd = K
    return p


@pytest.mark.parametrize("K,T,every", [(3, 64, 16), (1, 64, 16), (1, 50, 7), (2, 64, 8), (5, 24, 10), (4, 30, 1), (3, 40, 40)])
def test_bound(K, T, every):
    from paper_2002_00250_amd.adjoint import GmmWindow
    H, W = 480, 640
    warm = GmmWindow(2, 8, 8, _params(K))     # (the library's own first allocations)
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    win = GmmWindow(T, H, W, _params(K), every)
    took = free - torch.cuda.mem_get_info()[0]
    segments = -(-T // min(every, T))
    asked = H * W * (8 * T + 24 * K * (segments + min(every, T)))
    win.close()
    warm.close()
    assert took <= asked + (16 << 20), (took, asked)  # (block sums, the allocator's granularity, a queue)


# T frames and K Gaussians: one segment, two with a short first one, several, segments of one frame
PLANS = [(1, 20, 20), (1, 20, 3), (1, 21, 1), (1, 5, 5), (2, 23, 4), (2, 90, 9), (3, 64, 16), (3, 33, 8), (4, 60, 5),
         (5, 90, 9), (5, 3, 1), (3, 1, 1)]


@pytest.mark.parametrize("K,T,every", PLANS)
@pytest.mark.parametrize("H,W", [(9, 31), (365, 363)])
def test_plans_agree(K, T, every, H, W):
    from paper_2002_00250_amd.adjoint import GmmWindow
    if H > 9 and T > 40:
        T = 40
    g = torch.Generator(device="cuda").manual_seed(K * T)
    base = torch.randint(0, 256, (H, W, 3), device="cuda", generator=g)
    rgb = (base + torch.randint(-40, 41, (T, H, W, 3), device="cuda", generator=g)).clamp(0, 255).to(torch.uint8)
    dep = torch.randint(-400, 4000, (T, H, W), device="cuda", generator=g).clamp(min=0).to(torch.int16)
    dZ = torch.randn((T, H, W), device="cuda", generator=g)
    theta = torch.tensor([0.05, 2.5, 1.0], device="cuda")
    whole = GmmWindow(T, H, W, _params(K), T + 1)     # enough for every frame
    Z, has = whole.forward(theta, rgb, dep)
    grad, rec = whole.backward(theta, rgb, dep, dZ), whole.records()
    win = GmmWindow(T, H, W, _params(K), every)
    for _ in range(2):
        z, h = win.forward(theta, rgb, dep)
        assert torch.equal(z, Z) and torch.equal(h, has) and np.array_equal(win.records(), rec)
        for _ in range(3):                            # the first uses what the forward kept, the others replay
            assert torch.equal(win.backward(theta, rgb, dep, dZ), grad)
    whole.close()
    win.close()


@pytest.mark.parametrize("K,T,every", [(3, 64, 16), (1, 20, 3)])
def test_backward_alone_in_a_captured_graph(K, T, every):
    from paper_2002_00250_amd.adjoint import GmmWindow
    H, W = 20, 37
    g = torch.Generator(device="cuda").manual_seed(2)
    rgb = torch.randint(90, 120, (T, H, W, 3), dtype=torch.uint8, device="cuda", generator=g)
    dep = torch.randint(1000, 1100, (T, H, W), device="cuda", generator=g).to(torch.int16)
    dZ = torch.randn((T, H, W), device="cuda", generator=g)
    theta = torch.tensor([0.05, 2.5, 1.0], device="cuda")
    win = GmmWindow(T, H, W, _params(K), every)
    win.forward(theta, rgb, dep)
    grad = win.backward(theta, rgb, dep, dZ)
    win.forward(theta, rgb, dep)                      # kept again when the capture begins
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out = win.backward(theta, rgb, dep, dZ)
    for i in range(4):
        out.zero_()
        graph.replay()
        assert torch.equal(out, grad), i
        if i == 1:
            win.forward(theta, rgb, dep)
        torch.cuda.synchronize()
    win.close()
