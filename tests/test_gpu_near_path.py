"""The near field's path as the context reports it: the comparisons of
transforms with table sums compare two different things."""
import pytest
import test_gpu_conv as conv

import paper_1503_08509_amd as fp

pytestmark = pytest.mark.gpu


def _path(n, **kw):
    st = fp.Context(1.0, 100, n, **kw).stats()
    assert st["near_fft"] == (st["near_path"] == fp.NEAR_PATH_FFT)
    return st["near_path"]


@pytest.mark.parametrize("n,q,support,nsr", conv.test_transforms_equal_table_sums.pytestmark[0].args[1])
def test_periodic_lattices_take_the_transforms(n, q, support, nsr):
    kw = dict(q=q, support=fp._SUPPORTS[support], n_sr=nsr, solver=fp.SOLVER_FDM)
    assert _path(n, **kw) == fp.NEAR_PATH_LATTICE
    assert _path(n, near_field=fp.NEAR_DIRECT, **kw) == fp.NEAR_PATH_SUMS


@pytest.mark.parametrize("n,q,nsr,bc", conv.test_padded_lattice_of_the_boxes.pytestmark[0].args[1])
def test_boxes_take_the_transforms(n, q, nsr, bc):
    kw = dict(q=q, n_sr=nsr, solver=fp.SOLVER_FDM, boundary=getattr(fp, bc))
    assert _path(n, **kw) == fp.NEAR_PATH_LATTICE
    assert _path(n, near_field=fp.NEAR_DIRECT, **kw) == fp.NEAR_PATH_SUMS


def test_other_paths():
    assert _path(8) == _path(16, near_field=fp.NEAR_FFT) == fp.NEAR_PATH_FFT
    assert _path(8, near_field=fp.NEAR_DIRECT) == fp.NEAR_PATH_SUMS
    assert _path(9, precision=fp.PRECISION_MIXED) == fp.NEAR_PATH_SUMS
    assert _path(66, q=2) == fp.NEAR_PATH_SUMS   # above 64 elements there is no plan


def test_static_storage_without_room_for_the_transforms():
    """20^3 elements fit the static storage, the transforms' arrays beside them do not; at 9^3 both do."""
    def path(n):
        c = fp.Context(1.0, 100, n, static=True)
        p = c.stats()["near_path"]
        c.close()
        return p
    assert path(20) == fp.NEAR_PATH_SUMS
    assert path(9) == fp.NEAR_PATH_LATTICE


@pytest.mark.parametrize("n,nb,path", [(16, 4, "LATTICE"), (16, 16, "SUMS")])
def test_batches_of_the_smallest_block(n, nb, path):
    """n_sr = 1: the table sums above 20000 elements in all (one-element q = 4), by transforms or sums the same result."""
    torch = pytest.importorskip("torch")
    import numpy as np

    rng = np.random.default_rng(nb)
    c, kw = 20, dict(q=4, n_sr=1, solver=fp.SOLVER_FDM)
    x = torch.from_numpy(rng.random((c * nb, 3))).cuda()
    Q = torch.from_numpy(np.tile(np.repeat([1.0, -1.0], c // 2), nb)).cuda()
    a, b = fp.Context(1.0, [c] * nb, n, **kw), fp.Context(1.0, [c] * nb, n, near_field=fp.NEAR_DIRECT, **kw)
    assert a.stats()["near_path"] == getattr(fp, "NEAR_PATH_" + path)
    oa, ob = (v.energy_forces(x, Q, dUdQ=True, Phi=True) for v in (a, b))
    for k in ("Phi", "F", "dUdQ"):
        assert float((oa[k] - ob[k]).norm() / ob[k].norm()) < conv.TOL
