"""The inverted file's lists and means: members in ascending order and their
FP32 sums in that order, on both transposition paths (few targets with many
entries each, and the general one), element by element."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def p():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2303_05455_amd as pkg
    return pkg


# 4096 entries and 16 to a target are the least of the path for few targets,
# 2048 targets its most; chunks of 4096 entries
@pytest.mark.parametrize("M,nlist", [(4095, 2), (4096, 2), (4096, 256), (4096, 257), (8193, 31), (32767, 2048), (32768, 2048),
                                     (40001, 2049), (65535, 4096),
                                     (65537, 4096), (70000, 4097)])
def test_means_are_sums_in_ascending_order(p, M, nlist):
    rng = np.random.default_rng(M + nlist)
    x = rng.normal(size=(M, 5)).astype(np.float32)
    xt = torch.as_tensor(x).cuda()
    c0, assign = p.ivhd_ivf_train(xt, nlist, 0)
    c1, _ = p.ivhd_ivf_train(xt, nlist, 1)
    c0, assign, c1 = c0.cpu().numpy(), assign.cpu().numpy(), c1.cpu().numpy()
    want = c0.copy()
    order = np.argsort(assign, kind="stable")
    ends = np.cumsum(np.bincount(assign, minlength=nlist))
    for c in range(nlist):
        rows = order[(ends[c - 1] if c else 0):ends[c]]
        if rows.size:   # cumsum adds one by one
            want[c] = np.cumsum(x[rows], axis=0, dtype=np.float32)[-1] * (np.float32(1) / np.float32(rows.size))
    assert np.array_equal(c1, want)
