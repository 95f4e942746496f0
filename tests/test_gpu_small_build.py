"""The one-block build at the edges of its sort (runs of 64, their merges), its
split lists and its moments (a tree that fits LDS and one that does not), node
by node against the oracle, as every build."""
import numpy as np
import pytest

from paper_1912_04197_amd import ics

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("leaf", [1, 16])
@pytest.mark.parametrize("n", [2, 63, 64, 65, 127, 129, 320, 1000, 1025, 2047, 3000, 4096])
def test_small_build(n, leaf):
    from paper_1912_04197_amd import api
    from test_gpu_parity import _check_tree, _clump

    ctx = api.Context(n, leaf_size=leaf)
    _check_tree(ctx, ics.plummer(n, seed=n), leaf, False)
    s = ics.rubble_pile(n, seed=n)
    s.mass[::3] = 0.0  # massless cells
    _check_tree(ctx, s, leaf, True)
    # equal keys (kept in index order) down a chain of single-child cells
    _check_tree(ctx, _clump(n, max(1, n // 3), seed=n), leaf, False)


def test_small_build_deep_pairs():
    """Every body has a close partner: each pair splits far down, so the levels
    hold as many splitting nodes as there can be (n / 2)."""
    from paper_1912_04197_amd import api
    from test_gpu_parity import _check_tree

    s = ics.uniform_cube(4096, seed=5)
    s.pos[1::2] = s.pos[::2] + 1e-5 * np.random.default_rng(5).standard_normal((2048, 3))
    _check_tree(api.Context(4096, leaf_size=1), s, 1, False)
