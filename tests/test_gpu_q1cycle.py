"""The one-launch cycle on the order-1 levels: meshes whose hierarchy enters it
at different levels and coarsens by 2 and 3, and every Chebyshev degree,
against the exact solver; a cycle that did less than a V-cycle would cost PCG
iterations, so those are held too."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    t = pytest.importorskip("torch")
    if not t.cuda.is_available():
        pytest.skip("needs a GPU")
    return t


def _charges(torch, N, seed):
    rng = np.random.default_rng(seed)
    return (torch.from_numpy(rng.random((N, 3))).cuda(),
            torch.from_numpy(rng.permutation(np.repeat([1.0, -1.0], N // 2))).cuda())


def _err(a, b):
    a, b = a.cpu().numpy(), b.cpu().numpy()
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


# first level of the cycle (and below): 8 (4); 9 (3); 10 (5); 12 (6, 3); 15 (5); 16 (8, 4); 18 (9, 3); 20 (10, 5);
# 12 below 24; 16 below 32 and 64; 18 below 36; 20 below 40; 7 and 13 have no such level
@pytest.mark.parametrize("n", [7, 8, 9, 10, 12, 13, 15, 16, 18, 20, 24, 32, 36, 40])
def test_solution_and_iterations(torch, n):
    import paper_1503_08509_amd as fp

    x, Q = _charges(torch, 600, n)
    b = fp.Context(1.0, 600, n, solver=fp.SOLVER_FDM)
    ob = b.energy_forces(x, Q, Phi=True)
    a = fp.Context(1.0, 600, n, mg_rtol=1e-13)
    oa = a.energy_forces(x, Q, Phi=True)
    # 1e-13 in the residual times the square root of the preconditioned condition number and the load's scaling
    assert _err(a.stage("phi"), b.stage("phi")) < 1e-9
    for k in ("Phi", "F"):
        assert _err(oa[k], ob[k]) < 1e-9
    # five V(3,3) iterations reach 1e-7 on every mesh; 13 digits take at most twice as many and two more
    assert a.stats()["mg_iterations"] <= 12
    c = fp.Context(1.0, 600, n)
    c.energy_forces(x, Q)
    assert c.stats()["mg_iterations"] <= 6


@pytest.mark.parametrize("deg", [1, 2, 4, 10])
def test_chebyshev_degrees(torch, deg):
    import paper_1503_08509_amd as fp

    counts = [60, 200, 40]
    parts = [_charges(torch, c, deg + c) for c in counts]
    x, Q = (torch.cat([p[k] for p in parts]) for k in (0, 1))
    oa, ob = (fp.Context(1.0, counts, 16, cheb_degree=deg, mg_rtol=1e-13, mg_max_iter=200, solver=s).energy_forces(
        x, Q, Phi=True) for s in (fp.SOLVER_MG, fp.SOLVER_FDM))
    for k in ("Phi", "F"):
        assert _err(oa[k], ob[k]) < 1e-9
