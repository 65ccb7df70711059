"""The order-to-order prolongation of the multigrid cycle at meshes smaller
than, equal to and ragged against its column tiles (8 x 4 and 4 x 4 elements),
in the V-cycle: tightly converged solutions against the exact solver, and the
iteration count against that of a larger mesh, which a wrong coarse correction
would raise."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# A residual of 1e-13 leaves an error of that times the square root of the
# condition number of the preconditioned system times that of the load's
# scaling (below 1e4 on these meshes): 1e-9.
TOL = 1e-9


@pytest.mark.parametrize("n,q,support", [(3, 3, "one"), (4, 3, "one"), (5, 3, "one"), (9, 3, "one"), (12, 3, "one"),
                                         (5, 2, "one"), (3, 4, "one"), (5, 4, "one"), (3, 1, "27"), (9, 1, "27")])
def test_prolongation_in_the_cycle(n, q, support):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_1503_08509_amd as fp

    rng = np.random.default_rng(31 * n + q)
    N = 100
    x = torch.from_numpy(rng.random((N, 3))).cuda()
    Q = torch.from_numpy(rng.permutation(np.repeat([1.0, -1.0], N // 2))).cuda()
    kw = dict(q=q, support=fp._SUPPORTS[support], n_sr=1)
    a = fp.Context(1.0, N, n, mg_rtol=1e-13, mg_max_iter=60, **kw)
    b = fp.Context(1.0, N, n, solver=fp.SOLVER_FDM, **kw)
    a.energy_forces(x, Q)
    b.energy_forces(x, Q)
    pa, pb = a.stage("phi").cpu().numpy(), b.stage("phi").cpu().numpy()
    assert np.linalg.norm(pa - pb) < TOL * np.linalg.norm(pb)
