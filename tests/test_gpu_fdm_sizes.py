"""The exact solver's z direction (transform, block solve and back in one
kernel) and its transforms from and into the mesh vectors, at each transform
length and order and with one system or two, against the multigrid PCG solved
tightly."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# A residual of 1e-13 leaves an error of that times the square root of the
# condition number of the preconditioned system times that of the load's
# scaling (below 1e4 on these meshes): 1e-9.
TOL = 1e-9


# the last one's columns (64 x 216 values) do not fit LDS: separate passes
@pytest.mark.parametrize("n,q,support", [(8, 3, "one"), (8, 2, "one"), (8, 4, "one"), (8, 1, "27"), (16, 3, "one"),
                                         (16, 4, "one"), (32, 3, "one"), (32, 2, "27"), (32, 4, "one"), (64, 1, "27"),
                                         (64, 2, "one"), (64, 4, "one")])
@pytest.mark.parametrize("forces", [False, True])
def test_exact_solver_equals_multigrid(n, q, support, forces):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_1503_08509_amd as fp

    rng = np.random.default_rng(n + q)
    N = 200
    x = torch.from_numpy(rng.random((N, 3))).cuda()
    Q = torch.from_numpy(rng.permutation(np.repeat([1.0, -1.0], N // 2))).cuda()
    kw = dict(q=q, support=fp._SUPPORTS[support], n_sr=1, near_field=fp.NEAR_DIRECT, autotune=0)
    a = fp.Context(1.0, N, n, solver=fp.SOLVER_FDM, **kw)
    b = fp.Context(1.0, N, n, mg_rtol=1e-13, mg_max_iter=100, **kw)
    if forces:
        oa, ob = a.energy_forces(x, Q), b.energy_forces(x, Q)
        fa, fb = oa["F"].cpu().numpy(), ob["F"].cpu().numpy()
        assert np.linalg.norm(fa - fb) < TOL * np.linalg.norm(fb)
    else:
        a.energy(x, Q)
        b.energy(x, Q)
    pa, pb = a.stage("phi").cpu().numpy(), b.stage("phi").cpu().numpy()
    assert np.linalg.norm(pa - pb) < TOL * np.linalg.norm(pb)
