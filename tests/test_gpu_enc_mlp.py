"""The encoder's fused forward pass against its layers as separate products.

The hidden activations are the same bits (the same products added in the same
order), so only the head's FP32 sums differ from the reference's FP64 ones: at
most gamma(h2 + 1) sum |h w| per coordinate, gamma(n) = n 2^-24 / (1 - n 2^-24),
plus one rounding of the bias sum."""
import numpy as np
import pytest

from oracle import mlp

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def pkg():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2303_05455_amd import api, parametric
    return api, parametric


def _value(bits):
    return (bits.cpu().numpy().astype(np.uint16).astype(np.uint32) << 16).view(np.float32).astype(np.float64)


# the row tiles of 32, 64, 96, 112 and 128 rows (8192, 16384, ... rows fill the
# CUs once), ragged; stages of 128 inputs and steps of 32 with tails; narrowest
# and widest layers
@pytest.mark.parametrize("rows,n_in,h1,h2", [
    (1, 8, 512, 512), (33, 32, 456, 512), (8192, 128, 512, 456), (8193, 136, 480, 512), (20000, 40, 512, 504),
    (27001, 784, 512, 512), (30000, 264, 504, 464), (127, 1024, 512, 512),
    # rows of any width and alignment: the last chunk of a row not whole
    (300, 9, 512, 512), (17, 100, 512, 512), (1, 131, 512, 512), (113, 255, 512, 512), (9000, 390, 512, 512)])
def test_fused_forward_matches_its_layers(pkg, rows, n_in, h1, h2):
    api, parametric = pkg
    rng = np.random.default_rng(rows + n_in)
    enc = parametric.ParametricIVHD(n_in, (h1, h2), seed=3, batch=64)
    p = enc.params()
    p = p + 0.05 * torch.as_tensor(rng.normal(size=p.numel()).astype(np.float32)).to(p.device)
    enc.set_params(p)
    x = rng.normal(size=(rows, n_in)).astype(np.float32)
    x16 = torch.from_numpy(mlp.bf16_bits(x).copy()).cuda()
    z = enc.embed(x16).cpu().numpy().astype(np.float64)

    at = np.cumsum([0, h1 * n_in, h1, h2 * h1, h2, 2 * h2, 2])
    w1, b1, w2, b2, w3, b3 = (p[at[i]:at[i + 1]].contiguous() for i in range(6))
    bits = [torch.from_numpy(mlp.bf16_bits(w.cpu().numpy()).copy()).cuda() for w in (w1, w2, w3)]
    a1 = api.ivhd_gemm_bf16(x16, bits[0], rows, h1, n_in, lda=n_in, ldb=n_in, trans_b=True, epilogue=1, bias=b1)
    a2 = api.ivhd_gemm_bf16(a1, bits[1], rows, h2, h1, lda=h1, ldb=h1, trans_b=True, epilogue=1, bias=b2)
    h, w = _value(a2), _value(bits[2]).reshape(2, h2)
    ref = h @ w.T + b3.cpu().numpy().astype(np.float64)
    n = (h2 + 1) * 2.0 ** -24
    bound = n / (1 - n) * (np.abs(h) @ np.abs(w).T) + 2.0 ** -23 * np.abs(ref)
    assert np.all(np.abs(z - ref) <= bound + 1e-30)
    enc.close()


# K-major operands with 16-byte rows: one row of k and tails of its steps of 32,
# ragged tiles of 256 x 128, every epilogue, split-K
@pytest.mark.parametrize("M,N,K,epi,splits", [
    (8, 8, 1, 0, 1), (256, 128, 33, 1, 1), (264, 136, 95, 2, 1), (16, 512, 64, 1, 1), (520, 640, 4097, 0, 7),
    (512, 784, 5001, 0, 32)])
def test_k_major_product_equals_the_one_of_transposed_copies(pkg, M, N, K, epi, splits):
    """The same terms in the same order on the K-contiguous path (its K padded
    with zeros to a multiple of 8, which adds nothing): equal bits."""
    api, _ = pkg
    rng = np.random.default_rng(M + N + K)
    a, b = (torch.from_numpy(mlp.bf16_bits(rng.normal(size=(K, w)).astype(np.float32)).copy()).cuda() for w in (M, N))
    bias = torch.as_tensor(rng.normal(size=N).astype(np.float32)).cuda() if epi == 1 else None
    mask = torch.from_numpy(mlp.bf16_bits(rng.normal(size=(M, N)).astype(np.float32)).copy()).cuda() if epi == 2 else None
    kw = dict(epilogue=epi, bias=bias, mask=mask, ldm=N if epi == 2 else 0, splits=splits)
    got = api.ivhd_gemm_bf16(a, b, M, N, K, lda=M, ldb=N, trans_a=True, **kw)
    Kp = (K + 7) // 8 * 8
    at, bt = (torch.zeros((w, Kp), dtype=torch.int16, device="cuda") for w in (M, N))
    at[:, :K] = a.T
    bt[:, :K] = b.T
    ref = api.ivhd_gemm_bf16(at, bt, M, N, Kp, lda=Kp, ldb=Kp, trans_b=True, **kw)
    assert torch.equal(got, ref)
