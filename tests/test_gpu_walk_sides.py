"""Opening decisions at the ends of the range of cell sides: a scene scaled by a power
of two opens the same nodes as long as the squares of its distances are numbers."""
import numpy as np
import pytest

from paper_1912_04197_amd import ics

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2000, 6000])
@pytest.mark.parametrize("scale", [-460, -480, 500, 509])
def test_counts_of_scaled_scenes(n, scale):
    from paper_1912_04197_amd.api import Context

    s = ics.uniform_ball(n, seed=n)
    up = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    ctx = Context(n, leaf_size=8, precision="fp64", counts=True)
    counts = []
    for k in (0, scale):
        ctx.compute_accel(up(np.ldexp(s.pos, k)), up(s.mass), 0.6, softening=0.0)
        counts.append(ctx.walk_counts(n).cpu().numpy())
    assert np.array_equal(*counts)


def test_root_square_beyond_the_range():
    """A root cube whose square is infinite (a side of 2^513): its cells' squares are
    numbers from level 2 on, and a body far from a small cluster accepts the cluster's
    nodes as an oracle that squares each level's side does."""
    import oracle
    from paper_1912_04197_amd.api import Context

    n = 3000
    s = ics.uniform_ball(n, seed=4)
    pos = np.ldexp(s.pos, 500)  # a ball of 2^500 beside one body 2^511 away
    pos[0] = [2.0 ** 511, 0.0, 0.0]
    pos[1] = [-(2.0 ** 512), 0.0, 0.0]
    up = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    ctx = Context(n, leaf_size=8, precision="fp64", counts=True)
    ctx.compute_accel(up(pos), up(s.mass), 0.6, softening=0.0)
    _, _, _, want = oracle.bh(pos, s.mass, 0.6, softening=0.0, leaf=8)
    assert np.array_equal(ctx.walk_counts(n).cpu().numpy(), want)
