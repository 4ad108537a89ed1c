"""The GMM step decides most comparisons on approximate values and falls back to the rounded
ones near a tie (gmm_device.h): from states made to sit on and next to every tie, masks and
states must equal the oracle's bit for bit.  Also the depth code and the frame addressing, whose
divisions are multiplications by host-made reciprocals, over their whole range."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from gpu_util import log, to_dev  # noqa: E402
from oracle.depth import upscale_nearest  # noqa: E402
from oracle.gmm import GmmParams, GmmRef  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2002_00250_amd import fgs
    fgs.lib()
    yield


def _fgs_params(p):
    from paper_2002_00250_amd import fgs
    c = fgs.fgs_gmm_params_default()
    c.Kc, c.Kd, c.lambda_, c.var_mode, c.rho_mode, c.w_depth = p.Kc, p.Kd, p.lam, p.var_mode, p.rho_mode, p.w_depth
    c.decision = p.decision
    return c


def _ulps(rng, x, most):
    """x moved by up to `most` float32 steps either way."""
    x = np.asarray(x, np.float32)
    return (x.view(np.int32) + rng.integers(-most, most + 1, x.shape).astype(np.int32)).view(np.float32)


def _mixture_near_ties(rng, K, C, V, X, lam2, H, W):
    """Weights, means and variances whose squared distances to X lie at lambda^2 and at each
    other, and whose rank keys lie at each other, within a few float32 steps; with unused
    Gaussians, vanishing weights and variances at the ends of the exponent range."""
    w = rng.uniform(0.05, 1.0, (K, H, W)).astype(np.float32)
    w = np.sort(w, axis=0)[::-1] / w.sum(0)
    v = rng.uniform(1.0, 700.0, (K, V, H, W)).astype(np.float32)
    mode = rng.integers(0, 8, (H, W))
    v = np.where(mode == 3, np.float32(1.0), v)                              # keys ordered by the weights alone
    w = np.where((mode == 3) & (np.arange(K)[:, None, None] > 0), _ulps(rng, np.broadcast_to(w[:1], w.shape), 2), w)
    far = 10.0 ** rng.uniform(-37, 37, (K, V, H, W))
    v = np.where(mode == 4, far.astype(np.float32), v)
    w = np.where((mode == 5) & (np.arange(K)[:, None, None] >= rng.integers(0, K, (H, W))), np.float32(0), w)
    w = np.where((mode == 6) & (np.arange(K)[:, None, None] == K - 1), (10.0 ** rng.uniform(-45, -30, (H, W))).astype(np.float32), w)
    # means at lambda standard deviations (modes 0, 1), all at one distance (2), or anywhere
    mu = rng.uniform(0, 255, (K, C, H, W)).astype(np.float32)
    s = np.sqrt(lam2 * v.sum(1) / (C if V == 1 else V)).astype(np.float32)
    at = (X[None] + s[:, None] * rng.choice([-1, 1], (K, C, H, W))).astype(np.float32)
    mu = np.where(mode <= 1, _ulps(rng, at, 2), mu)
    one = rng.uniform(0.1, 3.0, (H, W)) * np.sqrt(v.sum(1))
    mu = np.where(mode == 2, (X[None] + one[:, None]).astype(np.float32), mu)
    mu = np.where(mode == 7, X[None], mu)
    return w.astype(np.float32), mu.astype(np.float32), v.astype(np.float32)


CASES = {
    "K 3": GmmParams(Kc=3, Kd=3),
    "K 5": GmmParams(Kc=5, Kd=5),
    "K 7/3": GmmParams(Kc=7, Kd=3),
    "K 1": GmmParams(Kc=1, Kd=1),
    "per channel": GmmParams(Kc=3, Kd=3, var_mode=1, rho_mode=1),
    "density decision": GmmParams(Kc=3, Kd=3, decision=1),
    "lambda beyond the approximate range": GmmParams(Kc=3, Kd=3, lam=2.0e6),
}


@pytest.mark.parametrize("stream", [0, 1])
@pytest.mark.parametrize("name", list(CASES))
def test_decisions_at_ties(name, stream):
    from paper_2002_00250_amd import fgs
    p = CASES[name]
    H, W = 61, 117
    rng = np.random.default_rng(len(name) + 1000 * stream)
    rgb = rng.integers(0, 256, (H, W, 3)).astype(np.uint8)
    depth = rng.integers(0, 9000, (H, W)).astype(np.uint16)
    depth[rng.random((H, W)) < 0.1] = 0
    Xc = rgb.transpose(2, 0, 1).astype(np.float32)
    code = np.clip((255 * depth.astype(np.int64) + 5000) // 10000, 1, 255)
    Xd = np.where(depth > 0, code, 0).astype(np.float32)[None]
    lam2 = float(np.float32(p.lam) * np.float32(p.lam))
    V = 3 if p.var_mode else 1
    wc, mc, vc = _mixture_near_ties(rng, p.Kc, 3, V, Xc, min(lam2, 9.0), H, W)
    wd, md, vd = _mixture_near_ties(rng, p.Kd, 1, 1, Xd, min(lam2, 9.0), H, W)
    st = dict(w_c=wc, mu_c=mc, v_c=vc if p.var_mode else vc[:, 0], w_d=wd, mu_d=md[:, 0], v_d=vd[:, 0], t=1)
    ref = GmmRef(H, W, p)
    ref.set_state_planes(st)
    m = fgs.Model(fgs.FGS_GMM, H, W, _fgs_params(p))
    fgs.fgs_set_cache_policy(m.handle, fgs.FGS_CACHE_STREAM if stream else fgs.FGS_CACHE_KEEP)
    m.set_state(dict(st, algo=fgs.FGS_GMM, H=H, W=W, Kc=p.Kc, Kd=p.Kd))
    for t in range(3):
        with np.errstate(all="ignore"):
            want = ref.step(rgb, depth)
        m.push(*to_dev(rgb, depth))
        got = m.mask_host()
        diff = int((got != want).sum())
        g, r = m.state(), ref.state_planes()
        bad = {k: int((np.asarray(g[k], np.float32).view(np.uint32) != np.asarray(r[k], np.float32).view(np.uint32)).sum())
               for k in ("w_c", "mu_c", "v_c", "w_d", "mu_d", "v_d")}
        log(f"{name}, stream {stream}, frame {t}: mask diff {diff}, state {bad}, foreground {float((want > 0).mean()):.2f}")
        # (the density decision goes through exp, which is not correctly rounded)
        assert diff <= (1e-4 * H * W if p.decision else 0) and not any(bad.values())
    m.close()


@pytest.mark.parametrize("full_scale", [1, 2, 3, 255, 510, 9999, 10000, 65535, 65536, 16711425, 2**31 - 1])
def test_depth_codes_over_the_whole_range(full_scale):
    """Every 16-bit depth, read back from the first sample a PBAS model takes."""
    from paper_2002_00250_amd import fgs
    c = fgs.fgs_pbas_params_default()
    c.N, c.depth_max_mm = 2, full_scale
    m = fgs.Model(fgs.FGS_PBAS, 256, 256, c)
    depth = np.arange(65536, dtype=np.uint16).reshape(256, 256)
    m.push(*to_dev(np.zeros((256, 256, 3), np.uint8), depth))
    got = (m.state()["samples"][0] >> 24).reshape(-1)
    d = np.arange(65536, dtype=np.int64)
    want = np.where(d > 0, np.clip((255 * d + full_scale // 2) // full_scale, 1, 255), 0)
    m.close()
    assert np.array_equal(got, want)


@pytest.mark.parametrize("H,W,dH,dW,pad", [(1, 1, 0, 0, 0), (3, 70001, 0, 0, 5), (70001, 3, 0, 0, 2), (97, 255, 0, 0, 7),
                                           (50, 257, 33, 91, 3), (50, 257, 200, 400, 0), (1, 3000, 1, 2999, 1)])
def test_frame_addressing(H, W, dH, dW, pad):
    """Packed, strided and upscaled frames: the pixels a model takes."""
    from paper_2002_00250_amd import fgs
    rng = np.random.default_rng(H + W)
    rgb = rng.integers(0, 256, (H, W + pad, 3)).astype(np.uint8)
    depth = rng.integers(0, 65536, (dH or H, (dW or W) + pad)).astype(np.uint16)
    r, d = to_dev(rgb, depth)
    c = fgs.fgs_pbas_params_default()
    c.N = 2
    m = fgs.Model(fgs.FGS_PBAS, H, W, c)
    g = fgs.Model(fgs.FGS_GMM, H, W)
    for x in (m, g):
        x.push(r[:, :W], d[:, :dW or W])
    seen = np.ascontiguousarray(depth[:, :dW or W])
    if dH:
        seen = upscale_nearest(seen, H, W)
    d64 = seen.astype(np.int64)
    code = np.where(d64 > 0, np.clip((255 * d64 + 5000) // 10000, 1, 255), 0)
    want = rgb[:, :W].astype(np.uint32)
    want = want[..., 0] | want[..., 1] << 8 | want[..., 2] << 16 | code.astype(np.uint32) << 24
    st = g.state()
    assert np.array_equal(m.state()["samples"][0], want)
    assert np.array_equal(st["mu_c"][0].transpose(1, 2, 0), rgb[:, :W].astype(np.float32))
    assert np.array_equal(st["mu_d"][0][seen > 0], code[seen > 0].astype(np.float32))
    m.close()
    g.close()
