"""The scans of the evaluation kernels at their edges: neighbour lists and
ranks must equal the FP64 (distance, index) definition exactly, as both sides
decide them in FP64."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def p():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2303_05455_amd as pkg
    return pkg


def _points(M, N, kind, seed):
    rng = np.random.default_rng(seed)
    if kind == "outward":    # from row 0, each point is nearer than all before it: a cut at every tile
        Z = np.zeros((M, N), np.float32)
        Z[1:, 0] = np.arange(M - 1, 0, -1)
        return Z
    if kind == "same":       # all distances equal: the indices decide
        return np.full((M, N), 2.5, np.float32)
    if kind == "grid":
        return rng.integers(0, 3, size=(M, N)).astype(np.float32)
    return (rng.normal(size=(M, N)) * 10.0 ** rng.uniform(-3, 3, size=(M, 1))).astype(np.float32)


def _both(p, Z, rows, k, kc, seed):
    z = torch.as_tensor(Z).cuda()
    r = torch.as_tensor(rows).cuda()
    got = p.ivhd_eval_neighbours(z, r, k).cpu().numpy()
    cand = np.random.default_rng(seed).integers(0, Z.shape[0], size=(rows.size, kc)).astype(np.int32)
    return got, cand, p.ivhd_eval_ranks(z, r, torch.as_tensor(cand).cuda()).cpu().numpy()


# tiles of 256 candidates, chunks of 2048, 8 rows per block; 2, 8 and 16
# dimensions at a time; buffers of 320 places up to k = 31
@pytest.mark.parametrize("M,N,k,kc,Q,kind", [
    (2, 1, 1, 1, 2, "normal"), (256, 2, 31, 64, 9, "normal"), (257, 2, 32, 1, 8, "grid"), (4097, 2, 128, 5, 17, "normal"),
    (4100, 2, 100, 5, 16, "outward"), (4100, 2, 31, 5, 16, "outward"), (4100, 2, 128, 5, 8, "same"),
    (2050, 3, 20, 7, 7, "grid"), (2047, 8, 127, 3, 25, "normal"), (600, 8, 31, 9, 30, "same"),
    (513, 9, 31, 9, 30, "normal"), (3000, 16, 100, 64, 8, "grid"), (4200, 17, 10, 2, 11, "outward"),
    (1000, 33, 32, 6, 9, "same"), (1100, 64, 64, 6, 33, "normal")])
def test_scans_equal_the_rank_definition(p, M, N, k, kc, Q, kind):
    Z = _points(M, N, kind, seed=M + N)
    rows = np.concatenate([[0], np.sort(np.random.default_rng(k).choice(np.arange(1, M), Q - 1, replace=False))])
    rows = rows.astype(np.int32)
    got, cand, rank = _both(p, Z, rows, k, kc, seed=kc)
    assert np.array_equal(got, oracle.rank_neighbours(Z, k, rows))
    full = oracle._ranks_full(Z)
    assert np.array_equal(rank, full[rows[:, None], cand])


def test_scans_take_many_rows_in_bands(p):
    # 12,000 rows of 1024 dimensions are more than the scratch holds at once
    Z = _points(300, 1024, "normal", seed=1)
    rows = np.tile(np.arange(300, dtype=np.int32), 40)
    got, cand, rank = _both(p, Z, rows, 12, 4, seed=2)
    assert np.array_equal(got, oracle.rank_neighbours(Z, 12)[rows])
    assert np.array_equal(rank, oracle._ranks_full(Z)[rows[:, None], cand])


def test_points_that_are_not_finite_come_last_or_nowhere(p):
    """A pair without a finite distance is in no list (places without a pair
    hold INT32_MAX), and before no other pair."""
    Z = _points(300, 2, "normal", seed=3)
    Z[5, 0], Z[40, 1] = np.nan, np.inf
    rows = np.array([0, 5, 40, 299], np.int32)
    got, cand, rank = _both(p, Z, rows, 40, 3, seed=4)
    finite = np.flatnonzero(np.isfinite(Z).all(1))
    for q, r in ((0, 0), (3, 299)):
        at = int(np.flatnonzero(finite == r)[0])
        want = finite[oracle.rank_neighbours(Z[finite], 40, np.array([at], np.int32))[0]]
        assert np.array_equal(got[q], want)
    assert (got[1:3] == np.iinfo(np.int32).max).all()
    assert (rank[1] == 0).all()
