"""Device buffers that wait for the next object or call: results do not depend
on what used a buffer before, on which thread, or on which stream."""
import threading

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


def _work(p, M, seed, rounds=1):
    """A context, an edge plan and kNN calls of one size: their results."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    x = torch.randn((M, 24), generator=g, device="cuda")
    out = []
    for _ in range(rounds):
        nn = p.ivhd_knn_build(x, 3)
        y = torch.randn((M, 2), generator=torch.Generator(device="cuda").manual_seed(seed), device="cuda")
        ctx = p.Context(nn, y, rn=1, b=0.01, c=0.1, seed=seed, rn_resample_every=7)
        ctx.step(20)
        rows = torch.arange(0, M, 5, device="cuda", dtype=torch.int32)
        near = p.ivhd_eval_neighbours(y, rows, 8)
        out.append([t.cpu().numpy() for t in (nn, ctx.y, ctx.v, near)])
        ctx.close()
    return out


def test_threads_and_streams_do_not_share_buffers(p):
    sizes = [700, 2500, 700, 4100]   # two threads ask for the same classes
    want = [_work(p, M, 10 + t)[0] for t, M in enumerate(sizes)]
    got = [None] * len(sizes)

    def run(t):
        with torch.cuda.stream(torch.cuda.Stream()):
            got[t] = _work(p, sizes[t], 10 + t, rounds=4)

    threads = [threading.Thread(target=run, args=(t,)) for t in range(len(sizes))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for t in range(len(sizes)):
        assert got[t] is not None
        for again in got[t]:
            for a, b in zip(again, want[t]):
                assert np.array_equal(a, b)


def test_released_buffers_are_bounded(p):
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    _work(p, 900, 1)
    torch.cuda.empty_cache()
    free0 = torch.cuda.mem_get_info()[0]
    for M in (5000, 20000, 60000, 150000, 300000):
        nn = torch.stack([(torch.arange(M, device="cuda", dtype=torch.int32) + s) % M for s in range(1, 9)], 1)
        y = torch.zeros((M, 2), device="cuda")
        ctxs = [p.Context(nn.contiguous(), y, rn=2, b=0.01, c=0.1, seed=s) for s in range(6)]
        for c in ctxs:
            c.close()
        del nn, y
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    held = free0 - torch.cuda.mem_get_info()[0]
    # 512 MiB of waiting buffers, and what the runtime keeps for itself
    assert held <= (512 + 256) << 20
