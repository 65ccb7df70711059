"""The V-cycle enqueued before the residual is read: whether the guess that
another iteration follows holds or not, the outputs are those of a replayed
graph, which runs the same iterations and guesses nothing, bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mixed", [False, True])
@pytest.mark.parametrize("rtol", [0.5, 3e-2, 1e-3, 1e-4, 3e-6, 1e-7, 1e-8, 1e-11])
def test_same_iterations_as_a_replay(rtol, mixed):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_1503_08509_amd as fp

    rng = np.random.default_rng(8)
    N = 500
    x = torch.from_numpy(rng.random((N, 3))).cuda()
    Q = torch.from_numpy(rng.permutation(np.repeat([1.0, -1.0], N // 2))).cuda()
    kw = dict(mg_rtol=rtol, autotune=0)
    if mixed:
        kw["precision"] = 1
    eager = fp.Context(1.0, N, 8, **kw)
    graph = fp.Context(1.0, N, 8, use_graph=1, **kw)
    a = eager.energy_forces(x, Q, dUdQ=True, Phi=True)
    for _ in range(3):
        b = graph.energy_forces(x, Q, dUdQ=True, Phi=True)
    assert eager.stats()["mg_iterations"] == graph.stats()["mg_iterations"]
    for k in ("F", "dUdQ", "Phi"):
        assert torch.equal(a[k], b[k])
