"""Buckets too large for a block's LDS in sorts of more blocks than the GPU holds at
once: the order and keys equal those of a context's first build (passes over whole
keys), whatever the order in which the blocks run."""
import numpy as np
import pytest

from paper_1912_04197_amd import ics

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [700001, (1 << 21) + 5])  # 256- and 1024-thread blocks
def test_oversized_buckets(n):
    from paper_1912_04197_amd import api
    from test_gpu_parity import _dev

    s = ics.uniform_cube(n, seed=31)
    mass = _dev(s.mass)
    knots = s.pos.copy()
    rng = np.random.default_rng(32)
    # clusters far smaller than a bucket's cell, of 2000 to 40,000 bodies, all over
    # the cube; two of them in neighbouring cells
    at = np.concatenate([rng.uniform(-0.9, 0.9, (10, 3)), [[0.31, 0.31, 0.31], [0.31, 0.31, 0.33]]])
    first = 1
    for c, k in zip(at, np.geomspace(2000, 40000, len(at)).astype(int)):
        knots[first : first + k] = c * np.abs(s.pos).max() + 1e-6 * rng.standard_normal((k, 3))
        first += k
    ctx = api.Context(n, leaf_size=16)
    ctx.build_tree(_dev(s.pos), mass)  # an even scene: the next build sorts by buckets
    ctx.build_tree(_dev(knots), mass)
    got = ctx.tree()
    new = api.Context(n, leaf_size=16)
    new.build_tree(_dev(knots), mass)
    want = new.tree()
    assert torch.equal(got.order, want.order) and torch.equal(got.keys, want.keys)
