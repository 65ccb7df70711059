"""Forces by the transforms are as exact as by the table sums: their
difference stays at the rounding of the node fields, not above it."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# Both sides round the node fields to about 1e-15 of their size; the tables of the direct side miss their
# symmetry by up to 1.2e-14 of their largest entry (tests/test_host_symmetry.py bounds it).  The derivative of
# the basis across an element and the forces' own size give a factor below 4: 6e-14.  With tables that are not
# symmetric behind the octant's spectrum, and its angles rounded to float64, the difference is 1.4e-13 to 2.5e-13.
TOL = 6e-14


@pytest.mark.parametrize("n,q,support", [(9, 2, "one"), (12, 2, "27"), (11, 4, "one")])
def test_forces_of_transforms_and_table_sums(n, q, support):
    torch = pytest.importorskip("torch")
    import paper_1503_08509_amd as fp

    rng = np.random.default_rng(n)
    N = 2000
    x = torch.from_numpy(rng.random((N, 3))).cuda()
    Q = torch.from_numpy(rng.permutation(np.repeat([1.0, -1.0], N // 2))).cuda()
    kw = dict(q=q, support=fp._SUPPORTS[support], solver=fp.SOLVER_FDM)
    F = []
    for near in (fp.NEAR_AUTO, fp.NEAR_DIRECT):
        c = fp.Context(1.0, N, n, near_field=near, **kw)
        c.energy(x, Q)   # then the adjoint solve by itself: the joint solve of both systems rounds otherwise
        F.append(c.backward(c.stats()["generation"])[0])
    assert float((F[0] - F[1]).norm() / F[1].norm()) < TOL
