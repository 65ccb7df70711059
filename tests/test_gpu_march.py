"""The marching mesh operator (orders 3 to 6) at the edges of its tiles: the
multigrid PCG, every mode of the operator and the fused restriction among its
steps, solved tightly against the exact solver, which does not use them."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# A residual of 1e-13 leaves an error of that times the square root of the
# condition number of the preconditioned system times that of the load's
# scaling (below 1e4 on these meshes): 1e-9.
TOL = 1e-9


@pytest.fixture(scope="module")
def torch():
    t = pytest.importorskip("torch")
    if not t.cuda.is_available():
        pytest.skip("needs a GPU")
    return t


def _err(a, b):
    a, b = a.cpu().numpy(), b.cpu().numpy()
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


# p = 5 (q = 3): 2 x 2 and 4 x 4 element tiles, whole and ragged along each
# axis, one to several elements per march; the p = 3 level below it in 4 x 4
# and (from 44) 8 x 4 tiles; p = 4, 6, 3 as the fine level of other screens
@pytest.mark.parametrize("n,q,support", [(7, 3, "one"), (8, 3, "one"), (11, 3, "one"), (13, 3, "one"), (16, 3, "one"),
                                         (18, 3, "one"), (27, 3, "one"), (44, 3, "one"), (9, 2, "one"),
                                         (14, 2, "27"), (7, 4, "one"), (10, 4, "one"), (11, 1, "27"), (44, 1, "27")])
def test_multigrid_equals_exact_solver(torch, n, q, support):
    import paper_1503_08509_amd as fp

    rng = np.random.default_rng(100 * n + q)
    N = 400
    x = torch.from_numpy(rng.random((N, 3))).cuda()
    Q = torch.from_numpy(rng.permutation(np.repeat([1.0, -1.0], N // 2))).cuda()
    kw = dict(q=q, support=fp._SUPPORTS[support])
    a = fp.Context(1.0, N, n, mg_rtol=1e-13, mg_max_iter=200, **kw)
    b = fp.Context(1.0, N, n, solver=fp.SOLVER_FDM, **kw)
    oa, ob = (c.energy_forces(x, Q, dUdQ=True, Phi=True) for c in (a, b))
    assert _err(a.stage("phi"), b.stage("phi")) < TOL
    for k in ("F", "dUdQ", "Phi"):
        assert _err(oa[k], ob[k]) < TOL


def test_batch_takes_its_own_tiles(torch):
    """A batch plans its tiles for all its systems: equal to single runs to rounding."""
    import paper_1503_08509_amd as fp

    rng = np.random.default_rng(5)
    counts = [40, 300, 120, 80, 60, 200, 100]
    x = torch.from_numpy(rng.random((sum(counts), 3))).cuda()
    Q = torch.cat([torch.from_numpy(rng.permutation(np.repeat([1.0, -1.0], c // 2))) for c in counts]).cuda()
    kw = dict(mg_rtol=1e-13, mg_max_iter=200)
    o = fp.Context(1.0, counts, 9, **kw).energy_forces(x, Q, dUdQ=True, Phi=True)
    at = 0
    for c in counts:
        s = fp.Context(1.0, c, 9, **kw).energy_forces(x[at:at + c], Q[at:at + c], dUdQ=True, Phi=True)
        for k in ("F", "dUdQ", "Phi"):
            assert _err(o[k][at:at + c], s[k]) < TOL
        at += c
