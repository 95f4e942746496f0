"""Which sort ran: bh_sort_passes over the scenes that the sort's tests build, where the
level-5 flag of the statistics is the same for several sorts."""
import numpy as np
import pytest

from paper_1912_04197_amd import ics

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("leaf,n", [(8, 5000), (64, 9001), (4, 70000)])
def test_crowded_scenes(leaf, n):
    from paper_1912_04197_amd import api
    from test_gpu_parity import _dev
    from test_gpu_sort_passes import _crowd

    ctx = api.Context(n, leaf_size=leaf)
    spread, point = 0.9 / 32, 1e-5
    # each build sorts by what the one before it found
    for k, size, want in ((4000, spread, 0), (4000, spread, 3), (4000, point, 3), (4000, spread, 0),
                          (0, spread, 3)):
        s = _crowd(n, k, size, seed=k + want)
        ctx.build_tree(_dev(s.pos), _dev(s.mass))
        assert ctx.sort_passes() == want
    s = _crowd(n, 0, spread, 9)
    ctx.build_tree(_dev(s.pos), _dev(s.mass))
    assert ctx.sort_passes() in (2, 3) and ctx.stats()["bucket_sort"]
    s = ics.uniform_ball(4096, seed=1)
    ctx.build_tree(_dev(s.pos), _dev(s.mass))  # one block
    assert ctx.sort_passes() == 0


@pytest.mark.parametrize("per_node,want", [(23, 2), (25, 3)])
def test_third_pass(per_node, want):
    """512 level-5 cells of the diagonal blocks of a cube, evenly filled but one, with
    more bodies than a comparison takes."""
    from paper_1912_04197_amd import api
    from test_gpu_parity import _check_tree

    rng = np.random.default_rng(per_node)
    cells = np.stack(np.meshgrid(*[np.arange(0, 32, 4)] * 3), -1).reshape(-1, 3)
    cells[-1] = 31  # the cube's far corner
    pos = (np.repeat(cells, per_node, 0) + rng.random((512 * per_node, 3))) / 32
    pos[0], pos[-1] = 0.0, 1.0
    pos[1 : 1 + 40] = (cells[0] + rng.random((40, 3))) / 32
    s = ics.uniform_cube(len(pos), seed=1)
    s.pos[:] = pos
    ctx = api.Context(s.n, leaf_size=4)
    for k in range(3):
        _check_tree(ctx, s, 4, False)
        assert ctx.sort_passes() == (want if k else 0)


def test_no_third_pass_for_leaves_above():
    """A ball whose level-5 nodes are few (most bodies are in leaves of level 4) and small."""
    from paper_1912_04197_amd import api
    from test_gpu_parity import _dev

    s = ics.uniform_ball(20000, seed=20000)
    ctx = api.Context(s.n, leaf_size=16)
    for want in (0, 2, 2):
        ctx.build_tree(_dev(s.pos), _dev(s.mass))
        assert ctx.sort_passes() == want


def test_batch():
    from paper_1912_04197_amd import api
    from test_gpu_parity import _dev
    from test_gpu_sort_passes import _crowd

    sizes = (5000, 37, 4800, 4500)
    parts = [_crowd(k, min(k - 1, 4000), 0.9 / 32, 7 + k) for k in sizes]
    pos = _dev(np.concatenate([p.pos for p in parts]))
    mass = _dev(np.full(sum(sizes), 1.0 / 5000))
    off = np.concatenate([[0], np.cumsum(sizes)])
    ctx = api.Context(sum(sizes), leaf_size=8, max_scenes=4)
    for want in (0, 3, 3):
        ctx.batched_accel(off, pos, mass, theta=0.5, softening=1e-3)
        assert ctx.sort_passes() == want


def test_null_context():
    from paper_1912_04197_amd import _lib as L

    assert L.load().bh_sort_passes(None) == -1
