"""The kept events that order a model's stream with torch's current one: long work on either side is
waited for, also when an event is recorded again before earlier waits on it have run, on any
current stream, and inside a captured graph."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from oracle.gmm import GmmRef  # noqa: E402
from synth import Scene, preset  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2002_00250_amd import fgs
    fgs.lib()
    yield


H, W = 40, 56


def _frames(n):
    sc = Scene(preset("gmm_320x240", H=H, W=W))
    fr = [sc.frame(t)[:2] for t in range(n)]
    ref = GmmRef(H, W)
    return fr, [ref.step(*f) for f in fr]


@pytest.mark.parametrize("own_stream", [True, False])
@pytest.mark.parametrize("current", ["default", "side"])
def test_frames_made_and_masks_used_behind_long_work(own_stream, current):
    from paper_2002_00250_amd import fgs
    fr, want = _frames(8)
    side = torch.cuda.Stream()
    m = fgs.Model(fgs.FGS_GMM, H, W, stream=None if own_stream else side)
    src = [(torch.from_numpy(r).cuda(), torch.from_numpy(d.view(np.int16)).cuda()) for r, d in fr]
    rgb, dep = torch.zeros_like(src[0][0]), torch.zeros_like(src[0][1])
    got = torch.zeros((len(fr), H, W), dtype=torch.uint8, device="cuda")
    busy = torch.randn((2048, 2048), device="cuda")
    torch.cuda.synchronize()
    with torch.cuda.stream(side if current == "side" else torch.cuda.default_stream()):
        out = torch.empty((H, W), dtype=torch.uint8, device="cuda")
        for i, (r, d) in enumerate(src):
            for _ in range(4):
                busy = busy @ busy * 1e-4     # the frame is written only after this
            rgb.copy_(r)
            dep.copy_(d)
            m.push(rgb, dep)
            rgb.zero_()                       # and cleared once the model has read it
            dep.zero_()
            m.mask_into(out)
            got[i].copy_(out)
            out.zero_()
    torch.cuda.synchronize()
    assert np.array_equal(got.cpu().numpy(), np.stack(want))
    m.close()


def test_orders_of_many_calls_ahead_of_the_device():
    from paper_2002_00250_amd import fgs
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    o = fgs.StreamOrder(a.cuda_stream)
    x = torch.zeros(1 << 16, device="cuda")
    torch.cuda.synchronize()
    for _ in range(200):                      # increments that would be lost if the streams overlapped
        with torch.cuda.stream(b):
            x += 1
        o.enter(b)
        with torch.cuda.stream(a):
            x += 1
        o.leave(b)
    torch.cuda.synchronize()
    assert bool((x == 400).all())
    o.enter(a)                                # the stream itself: nothing to wait for
    o.close()
    o.close()


def test_push_in_a_captured_graph():
    from paper_2002_00250_amd import fgs
    fr, want = _frames(6)
    m = fgs.Model(fgs.FGS_GMM, H, W)
    rgb, dep = torch.zeros((H, W, 3), dtype=torch.uint8, device="cuda"), torch.zeros((H, W), dtype=torch.int16, device="cuda")
    out = torch.zeros((H, W), dtype=torch.uint8, device="cuda")
    rgb.copy_(torch.from_numpy(fr[0][0]))
    dep.copy_(torch.from_numpy(fr[0][1].view(np.int16)))
    m.push(rgb, dep)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        m.push(rgb, dep)
        m.mask_into(out)
    for (r, d), w in zip(fr[1:], want[1:]):
        rgb.copy_(torch.from_numpy(r))
        dep.copy_(torch.from_numpy(d.view(np.int16)))
        g.replay()
        assert np.array_equal(out.cpu().numpy(), w)
        torch.cuda.synchronize()
    m.close()


def _dev(fr):
    return [(torch.from_numpy(r).cuda(), torch.from_numpy(d.view(np.int16)).cuda()) for r, d in fr]


@pytest.mark.parametrize("seen", [False, True])
def test_calls_from_many_streams_keep_the_models_order(seen):
    """Pushes, reads and counters from several streams, each behind long work on its own, with raw
    calls on the model's stream between: the model's calls run in the order they were made."""
    from paper_2002_00250_amd import fgs
    fr, want = _frames(24)
    src = _dev(fr)
    gt = (torch.rand((H, W), device="cuda") < 0.5).to(torch.uint8)
    m = fgs.Model(fgs.FGS_GMM, H, W)
    if seen:
        assert m.stream_handle
    streams = [torch.cuda.default_stream(), torch.cuda.Stream(), torch.cuda.Stream()]
    busy = [torch.randn((1024, 1024), device="cuda") for _ in streams]
    outs = torch.zeros((len(fr), H, W), dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    counts = np.zeros(4, np.int64)
    g = gt.cpu().numpy() != 0
    for i, (r, d) in enumerate(src):
        k = (i * 7) % 4
        if k == 3:                                # a raw call, on the model's own stream
            fgs.fgs_push_frame(m.handle, r.data_ptr(), r.stride(0), d.data_ptr(), 2 * d.stride(0), fgs.FGS_MEM_DEVICE)
        else:
            with torch.cuda.stream(streams[k]):
                for _ in range(6):
                    busy[k] = busy[k] @ busy[k] * 1e-3
                m.push(r, d)
        with torch.cuda.stream(streams[(i * 5) % 3]):
            m.eval_accumulate(gt)
            m.mask_into(outs[i])
        w = want[i] != 0
        counts += [(w & g).sum(), (~w & ~g).sum(), (w & ~g).sum(), (~w & g).sum()]
        if i % 8 == 5:
            assert np.array_equal(m.mask_host(), want[i])
        if i % 8 == 6:
            assert m.state()["t"] == i + 1
    assert m.eval_read(reset=True) == tuple(int(c) for c in counts)
    torch.cuda.synchronize()
    assert np.array_equal(outs.cpu().numpy(), np.stack(want))
    ref = GmmRef(H, W)
    for f in fr:
        ref.step(*f)
    st = m.state()
    for key, v in ref.state_planes().items():
        if key != "t":
            assert np.array_equal(st[key], v), key
    m.close()


def test_the_stream_handle_covers_earlier_and_later_work():
    """A caller that asks for the model's stream can wait for the model there, also for work that
    ran elsewhere before it asked, and fgs_sync and destruction wait for it."""
    from paper_2002_00250_amd import fgs
    fr, want = _frames(6)
    src = _dev(fr)
    busy = torch.randn((2048, 2048), device="cuda")
    m = fgs.Model(fgs.FGS_GMM, H, W)
    side = torch.cuda.Stream()
    torch.cuda.synchronize()

    def behind_busy(i):
        nonlocal busy
        with torch.cuda.stream(side):
            for _ in range(6):
                busy = busy @ busy * 1e-4
            m.push(*src[i])

    out = np.zeros((H, W), np.uint8)
    behind_busy(0)
    m.sync()
    assert side.query()
    behind_busy(1)
    ext = torch.cuda.ExternalStream(m.stream_handle)
    ext.synchronize()
    assert side.query()
    for i in (2, 3, 4):
        behind_busy(i)
        ext.synchronize()                         # (the push runs on the handed-out stream now)
        fgs.fgs_get_mask(m.handle, out.ctypes.data, W, fgs.FGS_MEM_HOST)
        assert np.array_equal(out, want[i])
    m.close()
    n = fgs.Model(fgs.FGS_GMM, H, W)
    with torch.cuda.stream(side):
        for _ in range(6):
            busy = busy @ busy * 1e-4
        n.push(*src[0])
    n.close()                                     # frees the model's memory: only after the push
    assert side.query()


def test_errors_leave_the_order_as_it_was():
    from paper_2002_00250_amd import fgs
    fr, want = _frames(3)
    src = _dev(fr)
    m = fgs.Model(fgs.FGS_GMM, H, W)
    cur = torch.cuda.current_stream().cuda_stream
    with pytest.raises(fgs.FgsError) as e:
        fgs.fgs_get_mask_on(m.handle, src[0][0].data_ptr(), W, cur)
    assert e.value.status == fgs.FGS_ERR_BAD_STATE
    for i, (r, d) in enumerate(src):
        with pytest.raises(fgs.FgsError) as e:
            fgs.fgs_push_frame_on(m.handle, r.data_ptr(), 3 * W - 1, d.data_ptr(), 2 * W, H, W, cur)
        assert e.value.status == fgs.FGS_ERR_INVALID_ARG
        m.push(r, d)
        with pytest.raises(fgs.FgsError):
            fgs.fgs_eval_accumulate_on(m.handle, 0, W, cur)
        assert np.array_equal(m.mask_host(), want[i])
    m.close()
