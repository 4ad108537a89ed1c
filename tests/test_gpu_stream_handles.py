"""Handles that stand for more than one stream: hipStreamPerThread, one handle for a stream of each
thread, and a stream made again where a destroyed one was.  A model's calls run in the order they
were made, also where the handle of one call equals that of the call before."""
import ctypes
import threading

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from oracle.gmm import GmmRef  # noqa: E402
from synth import Scene, preset  # noqa: E402

H, W = 40, 56
PER_THREAD = 2                                # hipStreamPerThread


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2002_00250_amd import fgs
    fgs.lib()
    yield


def _case(n):
    sc = Scene(preset("gmm_320x240", H=H, W=W))
    fr = [sc.frame(t)[:2] for t in range(n)]
    ref = GmmRef(H, W)
    want = [ref.step(*f) for f in fr]
    src = [(torch.from_numpy(r).cuda(), torch.from_numpy(d.view(np.int16)).cuda()) for r, d in fr]
    out = torch.zeros((n, H, W), dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    return src, out, np.stack(want)


def _push(m, src, out, stream):
    from paper_2002_00250_amd import fgs
    (r, d) = src
    with torch.cuda.stream(torch.cuda.ExternalStream(stream)):
        torch.cuda._sleep(5_000_000)          # the call's stream is busy when it is made
    fgs.fgs_push_frame_on(m.handle, r.data_ptr(), r.stride(0), d.data_ptr(), 2 * d.stride(0), H, W, stream)
    fgs.fgs_get_mask_on(m.handle, out.data_ptr(), W, stream)


def test_threads_in_turn_on_the_stream_of_each():
    from paper_2002_00250_amd import fgs
    src, out, want = _case(8)
    m = fgs.Model(fgs.FGS_GMM, H, W)
    failed = []
    turns = [threading.Semaphore(1), threading.Semaphore(0)]

    def thread(k):
        try:
            for i in range(k, len(src), 2):
                turns[k].acquire()            # (one thread at a time in the model)
                _push(m, src[i], out[i], PER_THREAD)
                turns[1 - k].release()
        except Exception as e:
            failed.append(e)
            turns[1 - k].release()

    threads = [threading.Thread(target=thread, args=(k,)) for k in (0, 1)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not failed, failed
    m.sync()
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy(), want)
    assert m.t == len(src)
    m.close()


def test_streams_made_and_destroyed_in_turn():
    from paper_2002_00250_amd import fgs
    hip = ctypes.CDLL("libamdhip64.so")
    src, out, want = _case(8)
    m = fgs.Model(fgs.FGS_GMM, H, W)
    for i, f in enumerate(src):
        s = ctypes.c_void_p()
        assert hip.hipStreamCreateWithFlags(ctypes.byref(s), 1) == 0
        _push(m, f, out[i], s.value)
        assert hip.hipStreamDestroy(s) == 0   # (its work is finished first, or later by itself)
    m.sync()
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy(), want)
    m.close()
