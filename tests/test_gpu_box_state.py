"""The box that a context keeps empty between builds, and the moments of the top
levels: builds of one context that go from wide scenes to narrow ones through every
kind of build, at the sizes where the chunks of the box reduction change. The tree
has to equal the oracle's, box included, so the bar is _check_tree's equality."""
import numpy as np
import pytest

from paper_1912_04197_amd import ics

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _wide(n, seed, size):
    """n bodies in a cube; the last one alone decides one side of the box."""
    s = ics.uniform_cube(n, seed=seed)
    s.pos *= size
    s.pos[-1, 0] = 3.0 * size
    return s


@pytest.mark.parametrize("leaf,n", [(64, 4097), (16, 5121), (1, 9000)])
def test_box_between_builds(leaf, n):
    from paper_1912_04197_amd import api
    from test_gpu_parity import _check_tree, _dev

    ctx = api.Context(n, leaf_size=leaf)
    # 4096 bodies and fewer: one block; the rest many launches
    for k, size, seed in ((n, 100.0, 1), (n, 1.0, 2), (900, 50.0, 3), (n, 0.5, 4), (4096, 7.0, 5),
                          (n, 0.25, 6)):
        _check_tree(ctx, _wide(k, seed, size), leaf, False)
    bad = _wide(n, 7, 1.0)
    bad.pos[n // 2, 1] = np.nan
    with pytest.raises(api.BHError):
        ctx.build_tree(_dev(bad.pos), _dev(bad.mass))
    _check_tree(ctx, _wide(n, 8, 0.125), leaf, False)


@pytest.mark.parametrize("n", [262144, 262145, 524289])
def test_box_chunks(n):
    from paper_1912_04197_amd import api
    from test_gpu_parity import _dev

    ctx = api.Context(n, leaf_size=16)
    for size, seed in ((10.0, 1), (1.0, 2)):
        s = _wide(n, seed, size)
        ctx.build_tree(_dev(s.pos), _dev(s.mass))
        assert ctx.tree().box[0:3] == s.pos.min(0).tolist()
        assert ctx.tree().box[6] == (s.pos.max(0) - s.pos.min(0)).max()


def test_box_scenes():
    """Batches of changing number of scenes, single bodies among them: every scene's
    forces equal those of a context that has seen nothing else."""
    from paper_1912_04197_amd import api
    from test_gpu_parity import _dev

    ctx = api.Context(12000, leaf_size=8, max_scenes=6)
    for sizes, scale, seed in (((3000, 1, 5000, 2, 700, 300), 30.0, 1), ((6000, 40), 1.0, 2),
                               ((10, 9000, 1), 0.1, 3)):
        s = _wide(sum(sizes), seed, scale)
        off = np.concatenate([[0], np.cumsum(sizes)])
        args = (_dev(s.pos), _dev(s.mass))
        got = ctx.batched_accel(off, *args, theta=0.5, softening=1e-3)
        new = api.Context(12000, leaf_size=8, max_scenes=6)
        want = new.batched_accel(off, *args, theta=0.5, softening=1e-3)
        got, want = (x[0] if isinstance(x, tuple) else x for x in (got, want))
        assert torch.equal(got, want)
