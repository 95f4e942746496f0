"""Launch hints of a build of another size: a large scene after a small one on one
context builds the oracle's tree, and no slower than on a context without hints."""
import numpy as np
import pytest

from paper_1912_04197_amd import ics

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def test_sizes_in_turn():
    from paper_1912_04197_amd import api
    from test_gpu_parity import _check_tree

    ctx = api.Context(60000, leaf_size=8)
    for k in (4500, 60000, 60000, 9000, 1000, 60000, 30000, 9001):
        _check_tree(ctx, ics.plummer(k, seed=k), 8, False)


def _build_ms(ctx, s):
    t = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    torch.cuda.synchronize()
    t[0].record()
    ctx.build_tree(*s, sync=False)
    t[1].record()
    torch.cuda.synchronize()
    return t[0].elapsed_time(t[1])


def test_large_after_small():
    """With a small scene's blocks for the subtrees of 2^20 bodies a build took twice as
    long as a first one without hints, with enough of them half as long."""
    from paper_1912_04197_amd import api

    up = lambda s: tuple(torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
                         for a in (s.pos, s.mass))
    small, large = up(ics.uniform_ball(5000, seed=1)), up(ics.uniform_ball(1 << 20, seed=2))
    first = min(_build_ms(api.Context(1 << 20, leaf_size=4), large) for _ in range(4))
    ctx = api.Context(1 << 20, leaf_size=4)
    after = []
    for _ in range(4):
        ctx.build_tree(*small)
        after.append(_build_ms(ctx, large))
    print(f"first {first:.3f} ms, after a small scene {min(after):.3f} ms")
    assert min(after) <= first
