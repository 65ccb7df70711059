"""The marching operator at order 3 on meshes smaller than its widest tile,
in batches large enough to ask for that tile."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# as in test_gpu_march.py: a residual of 1e-13 on a system of condition below 1e4
TOL = 1e-9


@pytest.mark.parametrize("n,nb,nsr,q,support", [(4, 1024, 1, 3, "one"), (4, 1024, 1, 1, "27"), (5, 700, 2, 3, "one")])
def test_batch_on_a_mesh_narrower_than_the_tile(n, nb, nsr, q, support):
    torch = pytest.importorskip("torch")
    import paper_1503_08509_amd as fp

    rng = np.random.default_rng(n * nb)
    c = 8
    x = torch.from_numpy(rng.random((c * nb, 3))).cuda()
    Q = torch.from_numpy(np.concatenate([rng.permutation(np.repeat([1.0, -1.0], c // 2)) for _ in range(nb)])).cuda()
    kw = dict(q=q, support=fp._SUPPORTS[support], n_sr=nsr, mg_rtol=1e-13, mg_max_iter=200)
    o = fp.Context(1.0, [c] * nb, n, **kw).energy_forces(x, Q, dUdQ=True, Phi=True)
    one = fp.Context(1.0, c, n, **kw)
    for b in (0, 1, nb // 2, nb - 1):   # the last one's vectors end their allocations
        s = slice(c * b, c * (b + 1))
        r = one.energy_forces(x[s].contiguous(), Q[s].contiguous(), dUdQ=True, Phi=True)
        for k in ("Phi", "F", "dUdQ"):
            d = (o[k][s] - r[k]).norm() / r[k].norm()
            assert float(d) < TOL, (b, k)
