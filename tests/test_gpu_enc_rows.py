"""The fused forward pass of more rows than one launch takes threads for."""
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def test_rows_beyond_one_launch():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2303_05455_amd import parametric
    enc = parametric.ParametricIVHD(8, (512, 512), seed=2, batch=64)
    base = 1 << 20
    x16 = parametric.ParametricIVHD.to_bf16(torch.randn((base, 8), device="cuda"))
    want = enc.embed(x16)
    rows = (1 << 30) + 5   # 2^23 blocks of 512 threads and one more
    big = torch.empty((rows, 8), dtype=torch.int16, device="cuda")   # 16 GiB
    for r in range(0, rows, base):
        big[r:r + base] = x16[:min(base, rows - r)]
    got = enc.embed(big)
    del big
    for r in range(0, rows, base):
        n = min(base, rows - r)
        assert torch.equal(got[r:r + n], want[:n]), r
