"""The boxes at the edges of their kernels' tiles: axes whose half (the number
of even modes) is a whole number of 16-mode tiles, one more, and odd and even;
a near block of more charges than one staging of the boundary values holds;
near blocks of one and two elements on a small mesh.  Against the oracle, with
the bounds of the other oracle comparisons of the boxes."""
import numpy as np
import pytest

import paper_1503_08509_amd as fp
from oracle import dirichlet as odir
from oracle import fep3m as ofe
from oracle import neumann as oneu

pytestmark = pytest.mark.gpu


# interior nodes per axis p n - 1 and box nodes p n + 1: 64 and 66 (13, q 3),
# 49 and 51 (10, q 3), 31 and 33 (8, q 2), 29 and 31 (6, q 3)
@pytest.mark.parametrize("kind", ["grounded", "insulated"])
@pytest.mark.parametrize("n,q,n_sr,corner", [(13, 3, 2, False), (10, 3, 3, False), (8, 2, 3, False), (6, 3, 1, False),
                                             (8, 3, 3, True)])
def test_box_tiles(kind, n, q, n_sr, corner):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    rng = np.random.default_rng(n + q)
    N = 1400 if corner else 150
    h = 1.0 / n
    x = rng.uniform(0.5 * h, 3.0 * h if corner else 1.0 - 0.5 * h, (N, 3))
    Q = rng.permutation(np.repeat([1.0, -1.0], N // 2))
    b = fp.BOUNDARY_GROUNDED if kind == "grounded" else fp.BOUNDARY_INSULATED
    ctx = fp.Context(1.0, N, n, q=q, n_sr=n_sr, boundary=b, solver=fp.SOLVER_FDM, table_box=2 * n_sr + 9)
    out = ctx.energy_forces(torch.from_numpy(x).cuda(), torch.from_numpy(Q).cuda(), dUdQ=True, Phi=True)
    ref = (odir if kind == "grounded" else oneu).energy_forces(x, Q, ofe.Params(L=1.0, n=n, q=q, n_sr=n_sr))
    for k in ("Phi", "F", "dUdQ"):
        a = out[k].cpu().numpy()
        assert np.linalg.norm(a - ref[k]) < 1e-10 * np.linalg.norm(ref[k]), k
