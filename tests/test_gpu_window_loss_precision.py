"""The loss of single scores: log(1 + exp(-x)) for a foreground pixel with x > 0, with nothing to
average its rounding away.  exp is off by up to an ulp (2^-23 of it at most, which the logarithm
passes on at most whole), the logarithm by 0.63 ulp: 1.63 x 2^-23 of the value."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def test_single_scores():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2002_00250_amd import fgs
    x = np.concatenate([np.linspace(1e-3, 4, 3000), np.linspace(4, 80, 1000)]).astype(np.float32)
    Z, n = torch.from_numpy(x).cuda(), x.size
    flag = torch.full((4,), 1, dtype=torch.uint8, device="cuda")
    loss, work = torch.empty(n, device="cuda"), torch.empty(fgs.FGS_WINDOW_BCE_WORK, dtype=torch.float64, device="cuda")
    s = torch.cuda.current_stream().cuda_stream
    for i in range(n):
        fgs.fgs_window_bce(Z.data_ptr() + 4 * i, flag.data_ptr(), flag.data_ptr(), 0, 1, 1.0, work.data_ptr(),
                           loss.data_ptr() + 4 * i, s)
    want = np.log1p(np.exp(-x.astype(np.float64)))
    off = np.abs(loss.cpu().numpy().astype(np.float64) - want) / want
    y = torch.nn.functional.binary_cross_entropy_with_logits(Z, torch.ones_like(Z), reduction="none")
    composed = np.abs(y.cpu().numpy().astype(np.float64) - want) / want
    print(f"largest error in 2^-23: {off.max() * 2 ** 23:.3f}, of the composed form {composed.max() * 2 ** 23:.3f}; "
          f"mean {off.mean() * 2 ** 23:.4f}, {composed.mean() * 2 ** 23:.4f}")
    assert off.max() <= 1.63 * 2.0 ** -23
