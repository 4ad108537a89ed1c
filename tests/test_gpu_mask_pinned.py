"""Masks read into host memory that the caller has pinned are copied there directly: in a fraction of the
time that pageable memory takes (a staging copy and one of the host; 1080x1920: 47 against 115 to 140 us); rows
that are not of whole words, where that copy goes row by row (7.7 ms), as fast as pageable ones."""
import time

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pad", [0, 32, 64, 1])
def test_rows_in_pinned_memory(pad):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2002_00250_amd import fgs
    H, W = 1080, 1920
    m = fgs.Model(fgs.FGS_GMM, H, W)
    rgb = torch.full((H, W, 3), 40, dtype=torch.uint8, device="cuda")
    depth = torch.full((H, W), 2000, dtype=torch.int16, device="cuda")
    m.push(rgb, depth)
    g = torch.Generator(device="cuda").manual_seed(3)
    fg = torch.rand((H, W), device="cuda", generator=g) < 0.4
    m.push(torch.where(fg[..., None], torch.full_like(rgb, 250), rgb), depth)
    want = fg.cpu().numpy() * np.uint8(255)
    pinned = torch.full((H, W + pad), 9, dtype=torch.uint8, pin_memory=True)
    plain = np.full((H, W + pad), 9, np.uint8)
    times = {}
    for name, ptr in (("plain", plain.ctypes.data), ("pinned", pinned.data_ptr())):
        t = []
        for _ in range(400):               # (a fresh pinned block may be slow for some 50 ms)
            a = time.perf_counter()
            fgs.fgs_get_mask(m.handle, ptr, W + pad, fgs.FGS_MEM_HOST)
            t.append(time.perf_counter() - a)
        times[name] = min(t)
    for out in (plain, pinned.numpy()):
        assert np.array_equal(out[:, :W], want) and (out[:, W:] == 9).all()
    print({k: round(v * 1e6, 1) for k, v in times.items()})
    assert times["pinned"] < (0.8 if pad % 4 == 0 else 1.5) * times["plain"], times
    m.close()
