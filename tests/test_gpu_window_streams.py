"""Frames made on another stream than the one a window is called on, and dropped right after the call:
their memory is not handed out again before the window's kernels have read it."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("direction", ["forward", "backward"])
def test_memory_of_frames_of_another_stream(direction):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2002_00250_amd.adjoint import GmmWindow
    T, H, W = 4, 96, 1024                     # 1.1 MiB of frames: blocks of their own
    g = torch.Generator(device="cuda").manual_seed(7)
    rgb = torch.randint(0, 256, (T, H, W, 3), dtype=torch.uint8, device="cuda", generator=g)
    dep = torch.randint(1, 4000, (T, H, W), device="cuda", generator=g).to(torch.int16)
    dZ = torch.randn((T, H, W), device="cuda", generator=g)
    theta = torch.tensor([0.05, 2.5, 1.0], device="cuda")
    win = GmmWindow(T, H, W)
    Z, _ = win.forward(theta, rgb, dep)
    grad = win.backward(theta, rgb, dep, dZ)
    maker, user = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()

    def make(x):
        with torch.cuda.stream(maker):
            return x.clone()

    probe = make(rgb)                         # (a block dropped unused is handed out again at once)
    at = probe.data_ptr()
    del probe
    probe = make(rgb)
    assert probe.data_ptr() == at
    del probe
    mine = [make(rgb), make(dep), make(dZ)]
    used = mine if direction == "backward" else mine[:2]
    ptrs = [x.data_ptr() for x in used]
    user.wait_stream(maker)
    with torch.cuda.stream(user):
        torch.cuda._sleep(100_000_000)        # the kernels wait behind this while the memory is dropped
        if direction == "forward":
            out, want = win.forward(theta, *used)[0], Z
        else:
            out, want = win.backward(theta, *used), grad
    kinds = [(tuple(x.shape), x.dtype) for x in used]
    del used, mine
    with torch.cuda.stream(maker):
        again = [torch.full(shape, 3, dtype=dtype, device="cuda") for shape, dtype in kinds]
    assert not user.query()                   # (still before the kernels)
    assert not set(ptrs) & {x.data_ptr() for x in again}
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy(), want.cpu().numpy())
    win.close()
