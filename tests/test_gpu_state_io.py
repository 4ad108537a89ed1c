"""State export and import at the edges of their kernels: widths around the 64x4 tile, sample
counts around the quads and words of slots, device blobs at an address that admits no 16-byte
access, neighbour writes still deferred, and headers that do not match.  All comparisons are of
bytes: the payload holds the model's numbers unchanged."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from gpu_util import to_dev  # noqa: E402
from synth import Scene, preset  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2002_00250_amd import fgs
    fgs.lib()
    yield


def _make(algo, H, W, kw):
    from paper_2002_00250_amd import fgs
    p = fgs.fgs_gmm_params_default() if algo == "gmm" else fgs.fgs_pbas_params_default()
    for k, v in kw.items():
        setattr(p, k, v)
    return fgs.Model(fgs.FGS_GMM if algo == "gmm" else fgs.FGS_PBAS, H, W, p)


def _frames(H, W, n):
    sc = Scene(preset("pbas_640x480", H=H, W=W))
    return [sc.frame(t)[:2] for t in range(n)]


def _device_blob(m, off):
    """The state in a device buffer at `off` bytes past an aligned address, guard bytes around it."""
    from paper_2002_00250_amd import fgs
    n = fgs.fgs_state_size(m.handle)
    buf = torch.full((n + 64,), 0x5A, dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    fgs.fgs_copy_state(m.handle, buf.data_ptr() + off, n, fgs.FGS_MEM_DEVICE)
    host = buf.cpu().numpy()
    assert (host[:off] == 0x5A).all() and (host[off + n:] == 0x5A).all()
    return buf, host[off:off + n]


CASES = [("pbas", 4, 64, dict(N=4)), ("pbas", 5, 65, dict(N=7)), ("pbas", 3, 63, dict(N=8)),
         ("pbas", 1, 1, dict(N=9)), ("pbas", 31, 130, dict(N=20)), ("pbas", 9, 67, dict(N=33)),
         ("pbas", 8, 192, dict(N=35)), ("pbas", 6, 70, dict(N=64)), ("pbas", 7, 45, dict(N=12, gradient=1)),
         ("gmm", 1, 1, dict(Kc=1, Kd=1)), ("gmm", 7, 37, dict(Kc=3, Kd=3, var_mode=1)),
         ("gmm", 16, 16, dict(Kc=7, Kd=3)), ("gmm", 13, 79, dict(Kc=7, Kd=3, var_mode=1))]


@pytest.mark.parametrize("off", [0, 4])
@pytest.mark.parametrize("algo,H,W,kw", CASES)
def test_round_trip(algo, H, W, kw, off):
    from paper_2002_00250_amd import fgs
    n = (kw.get("N", 4) + 6)
    frames = _frames(H, W, n + 4)
    a, flushed, b = (_make(algo, H, W, kw) for _ in range(3))
    for rgb, d in frames[:n]:
        a.push(*to_dev(rgb, d))
        flushed.push(*to_dev(rgb, d))
    fgs.fgs_get_state(flushed.handle)  # applies the deferred writes by themselves
    want = flushed.state_blob()
    buf, got = _device_blob(a, off)
    assert np.array_equal(got, want)
    assert np.array_equal(a.state_blob(), want)  # again, nothing deferred any more
    size = want.size
    b.push(*to_dev(*frames[0]))
    fgs.fgs_set_state(b.handle, buf.data_ptr() + off, size, fgs.FGS_MEM_DEVICE)
    assert b.t == n and np.array_equal(b.state_blob(), want)
    for rgb, d in frames[n:]:
        for m in (a, b, flushed):
            m.push(*to_dev(rgb, d))
    end = flushed.state_blob()
    assert np.array_equal(a.state_blob(), end) and np.array_equal(b.state_blob(), end)
    for m in (a, b, flushed):
        m.close()


def test_copy_settles_a_model_seen_in_place():
    """Addresses taken once hold the logical state after a later frame's fgs_copy_state too."""
    from paper_2002_00250_amd import fgs
    from test_gpu_state_fields import _values
    H, W, N = 9, 70, 20
    frames = _frames(H, W, N + 8)
    m = _make("pbas", H, W, dict(N=N))
    for rgb, d in frames[:-1]:
        m.push(*to_dev(rgb, d))
    fields = fgs.fgs_get_state(m.handle)
    m.push(*to_dev(*frames[-1]))
    st = m.state()
    for f in fields:
        if f["name"] == "samples":
            assert np.array_equal(_values(f, H, W), np.asarray(st["samples"])[f["index"]])
    m.close()


@pytest.mark.parametrize("algo,kw", [("pbas", dict(N=20)), ("pbas", dict(N=12, gradient=1)), ("gmm", dict(Kc=3, Kd=3))])
def test_device_header_that_does_not_match(algo, kw):
    """Refused as from the host, with the model as it was: its pending writes, its frames."""
    from paper_2002_00250_amd import fgs
    H, W = 11, 70
    n = kw.get("N", 4) + 5
    frames = _frames(H, W, n + 2)
    a, b = _make(algo, H, W, kw), _make(algo, H, W, kw)
    for rgb, d in frames[:n]:
        a.push(*to_dev(rgb, d))
        b.push(*to_dev(rgb, d))
    good = b.state_blob()
    words = [0, 1, 2, 3, 4, 5, 6, 7, 9] + ([10, 11] if algo == "pbas" else [])
    for w in words + ["frames"]:
        bad = good.copy().view(np.uint32)
        if w == "frames":
            bad[8] = 0xFFFFFFFF
        else:
            bad[w] ^= 1
        bad[16:] ^= 0x3C3C3C3C
        for where in ("host", "device"):
            if where == "device":
                t = torch.from_numpy(bad.view(np.int32).copy()).cuda()
                torch.cuda.synchronize()
                ptr, kind = t.data_ptr(), fgs.FGS_MEM_DEVICE
            else:
                ptr, kind = bad.ctypes.data, fgs.FGS_MEM_HOST
            with pytest.raises(fgs.FgsError) as e:
                fgs.fgs_set_state(a.handle, ptr, good.size, kind)
            assert e.value.status == fgs.FGS_ERR_INVALID_ARG
    assert a.t == n
    a.push(*to_dev(*frames[n]))
    b.push(*to_dev(*frames[n]))
    assert np.array_equal(a.state_blob(), b.state_blob())
    if algo == "gmm":  # a GMM state has no seed: those words do not matter
        other = good.copy().view(np.uint32)
        other[10] = 7
        t = torch.from_numpy(other.view(np.int32)).cuda()
        torch.cuda.synchronize()
        fgs.fgs_set_state(a.handle, t.data_ptr(), good.size, fgs.FGS_MEM_DEVICE)
        assert np.array_equal(a.state_blob(), good)
    a.close()
    b.close()
