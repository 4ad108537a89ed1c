"""A batched PBAS launch beyond three times the last-level cache (fewer workgroups per CU)
leaves the same model, byte for byte, as pushing each of its models alone."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,count,H,W", [(33, 4, 720, 1280), (64, 2, 700, 1203)])
def test_large_batch_equals_single_pushes(N, count, H, W):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2002_00250_amd import fgs
    assert count * H * W * N * 8 >= 768 << 20 > H * W * N * 8
    p = fgs.fgs_pbas_params_default()
    p.N = N
    stream = torch.cuda.Stream()
    batch, single = ([fgs.Model(fgs.FGS_PBAS, H, W, p, stream=stream) for _ in range(count)] for _ in range(2))
    g = torch.Generator(device="cuda").manual_seed(N)
    base = torch.randint(40, 200, (H, W, 3), device="cuda", generator=g, dtype=torch.int16)
    for t in range(N + 3):
        rgb = (base + torch.randint(-6, 7, (H, W, 3), device="cuda", generator=g, dtype=torch.int16)).to(torch.uint8)
        depth = torch.randint(0, 3000, (H, W), device="cuda", generator=g, dtype=torch.int16)
        fgs.push_frames(batch, [rgb] * count, [depth] * count)
        for m in single:
            m.push(rgb, depth)
    n = fgs.fgs_state_size(batch[0].handle)
    a, b = (torch.empty(n, dtype=torch.uint8, device="cuda") for _ in range(2))
    for x, y in zip(batch, single):
        torch.cuda.synchronize()
        fgs.fgs_copy_state(x.handle, a.data_ptr(), n, fgs.FGS_MEM_DEVICE)
        fgs.fgs_copy_state(y.handle, b.data_ptr(), n, fgs.FGS_MEM_DEVICE)
        assert torch.equal(a, b)
    for m in batch + single:
        m.close()
