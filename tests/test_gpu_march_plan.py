"""March lengths that suit the systems of a launch: the forward system solved
alone and together with the adjoint one takes the same steps bit for bit,
wherever the lengths differ, at orders 3 to 6.  The potentials then differ by
the gauge's constant alone, whose sum over the mesh is split over as many
blocks as the systems leave."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# One rounding of each potential (1 eps of the largest in all) and the
# constant: a mean of values up to that, whose sums of at most 2^9 terms per
# thread and tree above differ by at most a few eps.  Operators that differed
# in one rounding would be apart by the solver's amplification of it over five
# iterations, 1e-14 and more.
TOL = 16 * np.finfo(float).eps


@pytest.mark.parametrize("n,q,support", [(8, 3, "one"), (12, 3, "one"), (13, 3, "one"), (20, 3, "one"), (27, 3, "one"),
                                         (32, 3, "one"), (10, 2, "one"), (24, 2, "27"), (9, 4, "one"), (20, 1, "27"),
                                         (44, 1, "27")])
def test_same_steps_alone_or_together(n, q, support):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_1503_08509_amd as fp

    rng = np.random.default_rng(n + q)
    N = 200
    x = torch.from_numpy(rng.random((N, 3))).cuda()
    Q = torch.from_numpy(rng.permutation(np.repeat([1.0, -1.0], N // 2))).cuda()
    ctx = fp.Context(1.0, N, n, q=q, support=fp._SUPPORTS[support], n_sr=1, autotune=0)
    ctx.energy(x, Q)
    alone = ctx.stage("phi").clone()
    ctx.energy_forces(x, Q)
    both = ctx.stage("phi")
    assert float((both - alone).abs().max()) <= TOL * float(alone.abs().max())
