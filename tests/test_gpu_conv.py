"""Near field by transforms of lattices of any edge (near_field = AUTO) against
the table sums (DIRECT) on the same inputs: every radix the pass kernel has,
one and two factors, every screen family, near radii 1 to 3, the padded
lattices of the boxes, energies alone, backward after an energy-only forward."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# Both evaluate the same sums of at most 2744 (125 moments: 42875) products in
# float64, the transforms with up to 3 x 13 more additions per value; the
# result is a difference of mesh and near potentials up to 100 times larger
# (27-element q = 4): 1e-15 x sqrt(42875) x 100 < 1e-10.
TOL = 1e-10


@pytest.fixture(scope="module")
def torch():
    t = pytest.importorskip("torch")
    if not t.cuda.is_available():
        pytest.skip("needs a GPU")
    return t


def _charges(torch, N, n, seed, box):
    rng = np.random.default_rng(seed)
    x = rng.random((N, 3))
    if box:
        x = 0.5 / n + (1.0 - 1.0 / n) * x
    return (torch.from_numpy(x).cuda(), torch.from_numpy(rng.permutation(np.repeat([1.0, -1.0], N // 2))).cuda())


def _err(a, b):
    a, b = a.cpu().numpy(), b.cpu().numpy()
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


@pytest.mark.parametrize("n,q,support,nsr", [
    (7, 3, "one", 3), (9, 3, "one", 3), (10, 3, "one", 2), (11, 3, "one", 3), (12, 3, "one", 1), (13, 3, "one", 3),
    (14, 3, "one", 3), (15, 3, "one", 2), (18, 3, "one", 3), (20, 3, "one", 3), (22, 3, "one", 3), (26, 3, "one", 1),
    (27, 3, "one", 3), (30, 3, "one", 3), (63, 3, "one", 3), (8, 2, "one", 3), (9, 2, "one", 3), (8, 4, "one", 3),
    (11, 4, "one", 2), (16, 1, "27", 3), (9, 1, "27", 3), (8, 2, "27", 3), (12, 2, "27", 3), (7, 3, "27", 3),
    (16, 3, "27", 2), (8, 4, "27", 3)])
def test_transforms_equal_table_sums(torch, n, q, support, nsr):
    import paper_1503_08509_amd as fp

    x, Q = _charges(torch, 500, n, 10 * n + q, False)
    kw = dict(q=q, support=fp._SUPPORTS[support], n_sr=nsr, solver=fp.SOLVER_FDM)
    a, b = (fp.Context(1.0, 500, n, near_field=f, **kw) for f in (fp.NEAR_AUTO, fp.NEAR_DIRECT))
    oa, ob = (c.energy_forces(x, Q, dUdQ=True, Phi=True) for c in (a, b))
    for k in ("Phi", "F", "dUdQ"):
        assert _err(oa[k], ob[k]) < TOL, k
    # the moments' product alone, then the deposits' alone (both sides: the solver takes
    # phi and lambda one by one here, which differs from the joint solve by its own rounding)
    (Phi, _), (Pd, _) = a.energy(x, Q), b.energy(x, Q)
    assert _err(Phi, Pd) < TOL
    (F, g), (Fd, gd) = (c.backward(c.stats()["generation"]) for c in (a, b))
    assert _err(F, Fd) < TOL and _err(g, gd) < TOL


@pytest.mark.parametrize("n,q,nsr,bc", [(7, 3, 3, "BOUNDARY_GROUNDED"), (8, 2, 3, "BOUNDARY_GROUNDED"),
                                        (9, 4, 2, "BOUNDARY_INSULATED"), (11, 3, 1, "BOUNDARY_INSULATED"),
                                        (16, 3, 3, "BOUNDARY_GROUNDED"), (14, 3, 3, "BOUNDARY_INSULATED")])
def test_padded_lattice_of_the_boxes(torch, n, q, nsr, bc):
    import paper_1503_08509_amd as fp

    x, Q = _charges(torch, 300, n, n + q, True)
    kw = dict(q=q, n_sr=nsr, solver=fp.SOLVER_FDM, boundary=getattr(fp, bc))
    oa, ob = (fp.Context(1.0, 300, n, near_field=f, **kw).energy_forces(x, Q, dUdQ=True, Phi=True)
              for f in (fp.NEAR_AUTO, fp.NEAR_DIRECT))
    for k in ("Phi", "F", "dUdQ"):
        assert _err(oa[k], ob[k]) < TOL, k


def test_batch_and_charge_free_elements(torch):
    """Configurations of a batch share a block row of the products: each equals its own run."""
    import paper_1503_08509_amd as fp

    counts = [2, 90, 40]
    parts = [_charges(torch, c, 9, c, False) for c in counts]
    x, Q = (torch.cat([p[k] for p in parts]) for k in (0, 1))
    o = fp.Context(1.0, counts, 9, solver=fp.SOLVER_FDM).energy_forces(x, Q, dUdQ=True, Phi=True)
    at = 0
    for c, (xc, Qc) in zip(counts, parts):
        s = fp.Context(1.0, c, 9, solver=fp.SOLVER_FDM, near_field=fp.NEAR_DIRECT).energy_forces(xc, Qc, dUdQ=True, Phi=True)
        for k in ("Phi", "F", "dUdQ"):
            assert _err(o[k][at:at + c], s[k]) < TOL, (c, k)
        at += c
