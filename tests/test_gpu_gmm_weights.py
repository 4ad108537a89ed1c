"""The GMM step's weights (quotients by a shared reciprocal) and ranking (products in place of
keys) against the oracle bit for bit, in wavefronts that take the fast paths: a row of the frame
is one wavefront, and each kind of row holds weights, variances or rank keys near an edge of them."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from gpu_util import log, to_dev  # noqa: E402
from oracle.gmm import GmmParams, GmmRef  # noqa: E402
from test_gpu_gmm_decisions import _fgs_params  # noqa: E402

LOW = 2.0 ** -60  # the fast quotients' least weight
KINDS = ["ordinary", "wide", "edge in one lane", "subnormal in one lane", "unused", "keys apart by 2^-20 to 2^-14",
         "keys equal", "variances far apart", "one weight"]


def _mixture(rng, K, C, V, H):
    W = 64
    w = rng.uniform(0.05, 1.0, (K, H, W))
    v = rng.uniform(4.0, 700.0, (K, V, H, W))
    kind = np.arange(H) % len(KINDS)
    below = np.arange(K)[:, None, None] > 0
    row = lambda k: (kind == k)[None, :, None]  # noqa: E731
    lane = (np.arange(W)[None, None, :] == rng.integers(0, W, (1, H, 1)))
    w = np.where(row(1) & below, 10.0 ** rng.uniform(-17.9, 0, (K, H, W)), w)
    edge = LOW * (1 + rng.integers(-3, 4, (K, H, W)) * 2.0 ** -23) * 2.0 ** rng.integers(0, 2, (K, H, W))
    w = np.where(row(2) & below & lane, edge, w)
    w = np.where(row(3) & below & lane, 10.0 ** rng.uniform(-45, -37, (K, H, W)), w)
    w = np.where(row(4) & (np.arange(K)[:, None, None] >= rng.integers(1, K + 1, (1, H, W))), 0.0, w)
    w = -np.sort(-w, axis=0)
    w = w / w.sum(0)
    w = np.where(row(8) & below, 0.0, w)
    # a rank's variance such that its key follows the one above at the wanted distance
    vs = v.sum(1)
    for kd in (5, 6):
        for k in range(1, K):
            gap = 2.0 ** rng.uniform(-20, -14, (H, W)) * rng.choice([-1, 1], (H, W)) if kd == 5 else 0.0
            with np.errstate(all="ignore"):  # (rows of other kinds hold zeros)
                want = vs[k - 1] * (w[k] / w[k - 1]) ** 2 * (1 + gap)
            new = v[k] * (want / vs[k])[None]
            v[k] = np.where((kind == kd)[None, :, None], new, v[k])
            vs[k] = v[k].sum(0)
    v = np.where((kind == 7)[None, None, :, None], 10.0 ** rng.uniform(-18, 18, (K, 1, H, W)), v)
    mu = rng.uniform(0, 255, (K, C, H, W))
    return w.astype(np.float32), mu.astype(np.float32), v.astype(np.float32)


@pytest.mark.parametrize("Kc,Kd,var_mode", [(1, 1, 0), (2, 2, 0), (3, 3, 0), (5, 5, 0), (7, 3, 0), (3, 3, 1)])
def test_weights_and_ranking(Kc, Kd, var_mode):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2002_00250_amd import fgs
    H, W = 120 * len(KINDS), 64
    p = GmmParams(Kc=Kc, Kd=Kd, var_mode=var_mode)
    rng = np.random.default_rng(10 * Kc + Kd + var_mode)
    rgb = rng.integers(0, 256, (H, W, 3)).astype(np.uint8)
    depth = rng.integers(1, 9000, (H, W)).astype(np.uint16)
    wc, mc, vc = _mixture(rng, Kc, 3, 3 if var_mode else 1, H)
    wd, md, vd = _mixture(rng, Kd, 1, 1, H)
    st = dict(w_c=wc, mu_c=mc, v_c=vc if var_mode else vc[:, 0], w_d=wd, mu_d=md[:, 0], v_d=vd[:, 0], t=1)
    ref = GmmRef(H, W, p)
    ref.set_state_planes(st)
    m = fgs.Model(fgs.FGS_GMM, H, W, _fgs_params(p))
    m.set_state(dict(st, algo=fgs.FGS_GMM, H=H, W=W, Kc=Kc, Kd=Kd))
    for t in range(2):
        with np.errstate(all="ignore"):
            want = ref.step(rgb, depth)
        m.push(*to_dev(rgb, depth))
        g, r = m.state(), ref.state_planes()
        bad = {}
        for k in ("w_c", "mu_c", "v_c", "w_d", "mu_d", "v_d"):
            d = np.asarray(g[k], np.float32).view(np.uint32) != np.asarray(r[k], np.float32).view(np.uint32)
            rows = np.unique(np.nonzero(d)[-2])
            if rows.size:
                bad[k] = sorted({KINDS[i % len(KINDS)] for i in rows})
        log(f"K {Kc}/{Kd}, var_mode {var_mode}, frame {t}: not equal {bad}")
        assert not bad and np.array_equal(m.mask_host(), want)
    m.close()
