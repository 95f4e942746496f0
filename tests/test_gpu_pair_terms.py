"""Single FP64 pair terms against extended precision: scenes of two bodies, so that a
sum is one term.

Bar of a potential m / r with m = 1 and the offset along one axis: r^2 is one rounding
off (2^-54 in 1 / r), the residual of the estimate's square another (2^-54), the last
operation a third (2^-53): 2^-52 in all."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

ULP = 2.0 ** -52


@pytest.mark.parametrize("quad", [False, True])
def test_potential_of_a_pair(quad):
    from paper_1912_04197_amd import api

    k = 4000
    d = np.random.default_rng(5).uniform(0.5, 2.0, k)
    pos = np.zeros((2 * k, 3))
    pos[1::2, 0] = d
    ctx = api.Context(2 * k, leaf_size=8, precision="fp64", max_scenes=k, quad=quad)
    _, phi = ctx.batched_accel(np.arange(0, 2 * k + 1, 2), torch.from_numpy(pos).cuda(),
                               torch.ones(2 * k, dtype=torch.float64, device="cuda"), 0.5,
                               softening=0.0, potential=True)
    want = -1 / np.repeat(d, 2).astype(np.longdouble)
    err = np.abs((phi.cpu().numpy().astype(np.longdouble) - want) / want).max()
    print(f"worst {float(err) / ULP:.3f} ulp")
    assert err <= ULP
