"""Sorts by buckets of the top 24 key bits (scenes whose crowded part fills a level-5
cell but no level-8 cell), and the ways out of them: each build's tree equals the
oracle's, order and keys bit for bit, whatever the build before it promised."""
import numpy as np
import pytest

from paper_1912_04197_amd import ics

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _crowd(n, k, size, seed):
    """n bodies in a cube, k of them in a cube of `size` inside one level-5 cell."""
    s = ics.uniform_cube(n, seed=seed)
    rng = np.random.default_rng(seed)
    lo, ext = s.pos.min(0), (s.pos.max(0) - s.pos.min(0)).max()
    s.pos[1 : k + 1] = lo + ext * (11.05 / 32 + size * rng.random((k, 3)))
    return s


@pytest.mark.parametrize("leaf,n", [(8, 5000), (64, 9001), (4, 70000)])
def test_three_pass_buckets(leaf, n):
    from paper_1912_04197_amd import api
    from test_gpu_parity import _check_tree

    ctx = api.Context(n, leaf_size=leaf)
    spread, point = 0.9 / 32, 1e-5
    scenes = [_crowd(n, 4000, spread, 1),  # no hint yet
              _crowd(n, 4000, spread, 2),  # three passes
              _crowd(n, 4000, point, 3),   # three passes, one bucket too large for LDS
              _crowd(n, 4000, spread, 4),  # passes over whole keys
              _crowd(n, 0, spread, 5),     # three passes
              _crowd(n, 4000, spread, 6)]  # two passes
    for s in scenes:
        _check_tree(ctx, s, leaf, False)
        assert ctx.stats()["bucket_sort"] == (s is scenes[5])


@pytest.mark.parametrize("per_node", [23, 25])
def test_third_pass_for_many_bodies(per_node):
    """Either side of the mean number of bodies per level-5 node that takes a third
    pass: 512 level-5 cells of the diagonal blocks of a cube, evenly filled."""
    from paper_1912_04197_amd import api
    from test_gpu_parity import _check_tree

    rng = np.random.default_rng(per_node)
    cells = np.stack(np.meshgrid(*[np.arange(0, 32, 4)] * 3), -1).reshape(-1, 3)
    cells[-1] = 31  # the cube's far corner
    pos = (np.repeat(cells, per_node, 0) + rng.random((512 * per_node, 3))) / 32
    pos[0], pos[-1] = 0.0, 1.0
    s = ics.uniform_cube(len(pos), seed=1)
    s.pos[:] = pos
    ctx = api.Context(len(pos), leaf_size=4)
    for k in range(3):
        _check_tree(ctx, s, 4, False)
        assert ctx.stats()["bucket_sort"] == (k > 0)


def test_three_pass_buckets_batch():
    """Scenes of a batch sort by three passes and one on the scene index: the forces
    equal those of a context's first build (whole keys)."""
    from paper_1912_04197_amd import api
    from test_gpu_parity import _dev

    sizes = (5000, 37, 4800, 4500)
    parts = [_crowd(k, min(k - 1, 4000), 0.9 / 32, 7 + k) for k in sizes]
    pos = _dev(np.concatenate([p.pos for p in parts]))
    mass = _dev(np.full(sum(sizes), 1.0 / 5000))
    off = np.concatenate([[0], np.cumsum(sizes)])
    ctx = api.Context(sum(sizes), leaf_size=8, max_scenes=4)
    first = ctx.batched_accel(off, pos, mass, theta=0.5, softening=1e-3).clone()
    for _ in range(2):
        assert torch.equal(ctx.batched_accel(off, pos, mass, theta=0.5, softening=1e-3), first)
