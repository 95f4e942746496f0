"""Builds that make whole subtrees in one launch (the second and later builds of a
context, from the level that the previous build found small), node by node against
the oracle: even scenes, and scenes that break what the previous build promised -
one node of thousands of bodies below that level (long lists, searches, a chain to
the last level), then small nodes again."""
import numpy as np
import pytest

from paper_1912_04197_amd import ics

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _knot(n, k, size, seed):
    """n bodies in a cube, k of them within `size` of one point."""
    s = ics.uniform_cube(n, seed=seed)
    rng = np.random.default_rng(seed)
    s.pos[:k] = np.array([0.3, 0.1, -0.2]) + size * rng.standard_normal((k, 3))
    return s


@pytest.mark.parametrize("leaf,n", [(1, 9000), (4, 30000), (16, 5000), (64, 70000)])
def test_subtrees(leaf, n):
    from paper_1912_04197_amd import api
    from test_gpu_parity import _check_tree, _clump

    ctx = api.Context(n, leaf_size=leaf)
    even = ics.rubble_pile(n, seed=n)
    even.mass[::5] = 0.0
    scenes = [even, even, ics.plummer(n, seed=n), even,
              _knot(n, n - 500, 1e-4, seed=leaf),  # thousands of splitting nodes in one block
              even, _clump(n, n // 2, seed=leaf), even]
    for s in scenes:
        _check_tree(ctx, s, leaf, s is even)
