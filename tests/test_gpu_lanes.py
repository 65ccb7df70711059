"""Kernels that give several lanes to one element or charge, at counts that
leave waves and blocks partly filled: the pair count against a count on the
CPU, potentials and forces (the interpolation and the moment adjoint) against
the float64 oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    t = pytest.importorskip("torch")
    if not t.cuda.is_available():
        pytest.skip("needs a GPU")
    return t


@pytest.mark.parametrize("n,n_sr,counts", [(3, 1, 2), (5, 2, 31), (7, 3, 64), (8, 3, 65), (9, 1, [2, 34, 6]),
                                           (16, 2, 3000), (33, 3, 100)])
def test_pair_count(torch, n, n_sr, counts):
    import paper_1503_08509_amd as fp

    rng = np.random.default_rng(n)
    cs = counts if isinstance(counts, list) else [counts]
    x = rng.random((sum(cs), 3))
    Q = np.concatenate([np.r_[np.ones(c - c // 2) / (c - c // 2), -np.ones(c // 2) / (c // 2)] for c in cs])
    ctx = fp.Context(1.0, counts, n, n_sr=n_sr)
    ctx.energy(torch.from_numpy(x).cuda(), torch.from_numpy(Q).cuda())
    want, at = 0, 0
    for c in cs:
        e = np.minimum(np.floor(x[at:at + c] * n).astype(int), n - 1)
        d = np.abs(e[:, None] - e[None])
        d = np.minimum(d, n - d).max(axis=2)
        want += int((d <= n_sr).sum()) - c
        at += c
    assert ctx.stats()["near_pairs"] == want


# Charges that fill no wave, one wave but a lane and one block but a lane;
# n = 8 takes the transforms' moment adjoint.  The bounds are those of the
# oracle comparison at 1000 charges: solves to 1e-13, whose error the forces
# take on as 1e-9 and the potentials as 1e-10.
@pytest.mark.parametrize("N", [7, 33, 255, 257])
@pytest.mark.parametrize("n", [7, 8])
def test_potentials_and_forces_at_odd_counts(torch, N, n):
    import paper_1503_08509_amd as fp
    from oracle import adjoint, fep3m

    rng = np.random.default_rng(N + n)
    x = rng.random((N, 3))
    Q = rng.uniform(-1.0, 1.0, N)
    Q -= Q.mean()
    ref = adjoint.energy_forces(x, Q, fep3m.Params(L=1.0, n=n))
    ctx = fp.Context(1.0, N, n, mg_rtol=1e-13, mg_max_iter=100)
    out = ctx.energy_forces(torch.from_numpy(x).cuda(), torch.from_numpy(Q).cuda(), dUdQ=True, Phi=True)
    for k, tol in (("F", 1e-9), ("dUdQ", 1e-9), ("Phi", 1e-10)):
        a, b = out[k].cpu().numpy(), ref[k]
        assert np.linalg.norm(a - b) < tol * np.linalg.norm(b), k
