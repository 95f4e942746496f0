"""Upstream values that are not finite reach the gradients they are part of and no
others: a body's own upstream value has no part in its mass gradient."""
import numpy as np
import pytest

from paper_1912_04197_amd import ics

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("value", [float("nan"), float("inf")])
@pytest.mark.parametrize("theta", [0.0, 0.5])
@pytest.mark.parametrize("group", [16, 32, 64])
def test_own_mass_gradient(group, theta, value):
    from paper_1912_04197_amd.api import Context

    n, b = 5000, 1234
    s = ics.uniform_ball(n, seed=9)
    up = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    lam = np.random.default_rng(9).standard_normal((n, 3))
    ctx = Context(n, leaf_size=8, precision="fp64", adjoint=True, walk_group=group)
    out = []
    for v in (0.0, value):
        lam[b] = v
        out.append(ctx.accel_vjp(up(s.pos), up(s.mass), up(lam), theta=theta, softening=1e-2))
    (gp0, gm0), (gp, gm) = ([t.cpu().numpy() for t in o] for o in out)
    assert abs(gm[b] - gm0[b]) <= 1e-10 * np.abs(gm0).max()
    assert not np.isfinite(gp[b]).all()
    if theta == 0.0:  # every other body is one of its sources
        assert not np.isfinite(np.delete(gm, b)).any()
