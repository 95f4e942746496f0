"""The walk's queue between its traversing and evaluating waves where it can go
wrong: leaves of thousands of bodies (the queue runs far ahead of every batch),
one body or one batch in all, lists that end on either side of a batch, and
descriptors that fill the ring; forces, counts and force VJPs against the oracle
at the bars of their own tests (FP64 1e-12 A_i, FP32C 64u A_i, counts exact, VJPs
1e-10 of the largest component)."""
import numpy as np
import pytest

import oracle
from paper_1912_04197_amd import ics

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _clump(n, k):
    s = ics.uniform_ball(n, seed=n + k)
    s.pos[:k] = [0.1, -0.2, 0.3]
    return s


CASES = [
    # name, scene, leaf, theta
    ("clump6000", lambda: _clump(6000, 5000), 16, 0.5),  # one leaf of 5000 bodies
    ("pair", lambda: ics.uniform_ball(2, seed=2), 64, 0.5),
    ("batch", lambda: ics.uniform_ball(64, seed=3), 64, 0.5),
    ("batch_and_one", lambda: ics.uniform_ball(65, seed=4), 1, 0.0),
    ("one_body_leaves", lambda: ics.plummer(9000, seed=5), 1, 0.2),  # a descriptor an item
    ("big_leaves", lambda: ics.plummer(9001, seed=6), 64, 0.9),
]


@pytest.mark.parametrize("group", [16, 32, 64])
@pytest.mark.parametrize("name,make,leaf,theta", CASES, ids=[c[0] for c in CASES])
def test_walk_queue(name, make, leaf, theta, group):
    from paper_1912_04197_amd.api import Context

    s = make()
    up = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    ref, ref_phi, aabs, cnt = oracle.bh(s.pos, s.mass, theta, softening=1e-2, leaf=leaf)
    for precision, tol in (("fp64", 1e-12), ("fp32c", 64 * 2.0 ** -24)):
        ctx = Context(s.n, leaf_size=leaf, precision=precision, counts=True, walk_group=group)
        acc, phi = ctx.compute_accel(up(s.pos), up(s.mass), theta, softening=1e-2, potential=True)
        assert np.array_equal(ctx.walk_counts(s.n).cpu().numpy(), cnt)
        assert np.all(np.linalg.norm(acc.cpu().numpy() - ref, axis=1) <= tol * aabs + 1e-300)
        again = ctx.compute_accel(up(s.pos), up(s.mass), theta, softening=1e-2)
        assert torch.equal(again, acc)  # whichever wave was ahead
    lam = np.random.default_rng(9).standard_normal((s.n, 3))
    g_ref = oracle.tree_vjp(s.pos, s.mass, lam, theta, softening=1e-2, leaf=leaf)
    ctx = Context(s.n, leaf_size=leaf, precision="fp64", adjoint=True, walk_group=group)
    g = ctx.accel_vjp(up(s.pos), up(s.mass), up(lam), theta=theta, softening=1e-2)
    for a, r in zip(g, g_ref):
        assert np.abs(a.cpu().numpy() - r).max() <= 1e-10 * np.abs(r).max()
