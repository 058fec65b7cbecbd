"""Memory that waits inside the library goes back to the device on request."""
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def test_trim_gives_waiting_memory_back():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2303_05455_amd as p
    M = 1000000
    nn = torch.stack([(torch.arange(M, device="cuda", dtype=torch.int32) + s) % M for s in range(1, 6)], 1).contiguous()
    y = torch.randn((M, 2), device="cuda")

    def free():
        torch.cuda.synchronize()
        return torch.cuda.mem_get_info()[0]

    live = p.Context(nn, y.clone(), rn=1, b=1e-3, c=0.1, seed=3)
    gone = p.Context(nn, y.clone(), rn=1, b=1e-3, c=0.1, seed=3)
    p.ivhd_trim()
    before = free()
    gone.close()
    p.ivhd_trim()
    assert free() - before > 100 << 20   # its in- and out-lists alone: 4 x 20 MB, and 10 arrays of 8 MB
    live.step(5)
    again = p.Context(nn, y.clone(), rn=1, b=1e-3, c=0.1, seed=3)
    again.step(5)
    assert torch.equal(live.y, again.y)
    live.close()
    again.close()
