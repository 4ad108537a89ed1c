"""Reading the mask out: every alignment and stride of the destination, in device and host memory,
sizes around the copy's 16 bytes a lane, and images beyond the pinned staging."""
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


def _model(H, W, seed):
    """A model whose mask is a known speckle: one frame, then one that differs at random pixels."""
    from paper_2002_00250_amd import fgs
    g = torch.Generator(device="cuda").manual_seed(seed)
    m = fgs.Model(fgs.FGS_GMM, H, W)
    rgb = torch.full((H, W, 3), 40, dtype=torch.uint8, device="cuda")
    depth = torch.full((H, W), 2000, dtype=torch.int16, device="cuda")
    m.push(rgb, depth)
    fg = torch.rand((H, W), device="cuda", generator=g) < 0.4
    m.push(torch.where(fg[..., None], torch.full_like(rgb, 250), rgb), depth)
    want = (fg.to(torch.uint8) * 255).cpu().numpy()
    return m, want


@pytest.mark.parametrize("H,W", [(1, 1), (3, 5), (1, 15), (1, 16), (2, 17), (16, 16), (7, 33), (5, 64), (37, 255), (11, 1030)])
def test_every_alignment(H, W):
    from paper_2002_00250_amd import fgs
    m, want = _model(H, W, H * W)
    assert np.array_equal(m.mask_host(), want)
    for off, pad in ((0, 0), (0, 16), (1, 0), (2, 3), (4, 4), (8, 8), (3, 13), (16, 1)):
        stride = W + pad
        buf = torch.full((off + H * stride + 7,), 9, dtype=torch.uint8, device="cuda")
        torch.cuda.synchronize()
        fgs.fgs_get_mask(m.handle, buf.data_ptr() + off, stride, fgs.FGS_MEM_DEVICE)
        m.sync()
        host = np.full(off + H * stride + 7, 9, np.uint8)
        fgs.fgs_get_mask(m.handle, host.ctypes.data + off, stride, fgs.FGS_MEM_HOST)
        exp = np.full(off + H * stride + 7, 9, np.uint8)
        for y in range(H):
            exp[off + y * stride:off + y * stride + W] = want[y]
        assert np.array_equal(buf.cpu().numpy(), exp) and np.array_equal(host, exp), (off, pad)
    m.close()


@pytest.mark.parametrize("H,W,pad", [(4100, 4099, 0), (4100, 4099, 5), (2, (16 << 20) + 3, 1)])
def test_beyond_the_staging(H, W, pad):
    from paper_2002_00250_amd import fgs
    m, want = _model(H, W, 5)
    out = np.full((H, W + pad), 7, np.uint8)
    fgs.fgs_get_mask(m.handle, out.ctypes.data, W + pad, fgs.FGS_MEM_HOST)
    assert np.array_equal(out[:, :W], want) and (out[:, W:] == 7).all()
    m.close()


def test_destinations_the_kernel_leaves_to_the_runtime():
    """Pinned host memory named as device memory is written; rows past the end of an allocation
    are refused, not written."""
    from paper_2002_00250_amd import fgs
    H, W = 64, 96
    m, want = _model(H, W, 3)
    pinned = torch.zeros((H, W), dtype=torch.uint8, pin_memory=True)
    fgs.fgs_get_mask(m.handle, pinned.data_ptr(), W, fgs.FGS_MEM_HOST)
    assert np.array_equal(pinned.numpy(), want)
    pinned.zero_()
    fgs.fgs_get_mask(m.handle, pinned.data_ptr(), W, fgs.FGS_MEM_DEVICE)
    m.sync()
    assert np.array_equal(pinned.numpy(), want)
    m.close()


def test_push_and_read_from_the_host_in_turn():
    """Strided host frames and masks of one model, each read before the next push."""
    from paper_2002_00250_amd import fgs
    from oracle.gmm import GmmRef
    from synth import Scene, preset
    H, W = 45, 77
    sc = Scene(preset("gmm_320x240", H=H, W=W))
    ref, m = GmmRef(H, W), fgs.Model(fgs.FGS_GMM, H, W)
    for t in range(12):
        rgb, D, _ = sc.frame(t)
        want = ref.step(rgb, D)
        wide, deep = np.pad(rgb, ((0, 0), (0, t % 3), (0, 0))), np.pad(D, ((0, 0), (0, t % 4)))
        fgs.fgs_push_frame(m.handle, wide.ctypes.data, wide.strides[0], deep.ctypes.data, deep.strides[0], fgs.FGS_MEM_HOST)
        assert np.array_equal(m.mask_host(), want)
    m.close()
