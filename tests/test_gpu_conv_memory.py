"""Transforms whose arrays would take more than a quarter of the free device
memory are left to the table sums, and the context works beside them."""
import pytest

pytestmark = pytest.mark.gpu


def test_little_free_memory_takes_the_table_sums():
    torch = pytest.importorskip("torch")
    import paper_1503_08509_amd as fp

    n, N, kw = 40, 1000, dict(q=4, support=fp.SUPPORT_27, n_sr=2)
    x = torch.rand(N, 3, device="cuda", dtype=torch.float64, generator=torch.Generator("cuda").manual_seed(4))
    Q = 1.0 - 2.0 * (torch.arange(N, device="cuda") % 2).double()

    def held(**more):
        c = fp.Context(1.0, N, n, **kw, **more)
        st = c.stats()
        return c, st["device_bytes"], st["near_path"]

    c, sums, path = held(near_field=fp.NEAR_DIRECT)
    assert path == fp.NEAR_PATH_SUMS
    want = c.energy_forces(x, Q, dUdQ=True, Phi=True)
    c.close()
    c, both, path = held()
    assert path == fp.NEAR_PATH_LATTICE
    c.close()
    arrays = both - sums
    free, _ = torch.cuda.mem_get_info()
    keep = torch.empty(free - sums - 2 * arrays, dtype=torch.uint8, device="cuda")   # two arrays' worth left: half of the rule's
    try:
        c, now, path = held(use_graph=1)
        assert path == fp.NEAR_PATH_SUMS and now == sums
        for _ in range(2):   # the graph's buffers are allocated by the first call
            got = c.energy_forces(x, Q, dUdQ=True, Phi=True)
            for k in want:
                assert float((got[k] - want[k]).norm() / want[k].norm()) < 1e-12
        assert c.stats()["graph_replays"] == 1
        c.close()
    finally:
        del keep
        torch.cuda.empty_cache()
