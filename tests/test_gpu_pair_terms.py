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


SCALES = [
    # powers of two of lengths and masses: the term's factor m r^-3 would be infinite,
    # subnormal, or zero, the term m d r^-3 is not
    (-325, 60), (325, -60), (325, -150)]


@pytest.mark.parametrize("length,mass_scale", SCALES)
@pytest.mark.parametrize("n", [300, 1500, 4200])
def test_forces_at_the_edges_of_the_range(n, length, mass_scale):
    """Lengths times 2^a and masses times 2^b scale accelerations by 2^(b - 2 a) and
    potentials by 2^(b - a), exactly but for the rounding of each term (bar: that of
    every FP64 force, 1e-12 A_i; potentials the same relative to sum m / r)."""
    import oracle
    from paper_1912_04197_amd import api, ics

    s = ics.uniform_ball(n, seed=n)
    s.mass[::7] = 0.0
    up = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    _, ref_phi, aabs = oracle.direct(s.pos, s.mass)
    pos, mass = up(np.ldexp(s.pos, length)), up(np.ldexp(s.mass, mass_scale))
    ctx = api.Context(n, leaf_size=8, precision="fp64")
    for run in (lambda p, m: ctx.compute_accel_direct(p, m, potential=True),
                lambda p, m: ctx.compute_accel(p, m, 0.0, potential=True),
                lambda p, m: ctx.compute_accel(p, m, 0.6, potential=True)):
        acc, phi = (t.cpu().numpy() for t in run(up(s.pos), up(s.mass)))
        far, far_phi = (t.cpu().numpy() for t in run(pos, mass))
        far = np.ldexp(far, 2 * length - mass_scale)
        far_phi = np.ldexp(far_phi, length - mass_scale)
        assert np.all(np.linalg.norm(far - acc, axis=1) <= 1e-12 * aabs)
        assert np.all(np.abs(far_phi - phi) <= 1e-12 * np.abs(ref_phi))


@pytest.mark.parametrize("n", [300, 4200])
def test_one_extreme_body(n):
    """One body of a mass that leaves its terms' factors out of range among ordinary
    ones, and two bodies on one point: only their groups are summed pair by pair."""
    import oracle
    from paper_1912_04197_amd import api, ics

    s = ics.uniform_ball(n, seed=n + 1)
    s.mass[n // 2] = 1e-200
    s.pos[9] = s.pos[5]
    up = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    ref, ref_phi, aabs = oracle.direct(s.pos, s.mass)
    ctx = api.Context(n, leaf_size=8, precision="fp64")
    for run in (lambda: ctx.compute_accel_direct(up(s.pos), up(s.mass), potential=True),
                lambda: ctx.compute_accel(up(s.pos), up(s.mass), 0.0, potential=True)):
        acc, phi = (t.cpu().numpy() for t in run())
        assert np.all(np.linalg.norm(acc - ref, axis=1) <= 1e-12 * aabs)
        assert np.all(np.abs(phi - ref_phi) <= 1e-12 * np.abs(ref_phi))


@pytest.mark.parametrize("n", [200, 4200])
def test_offsets_beyond_the_range(n):
    """Two bodies so far out that their offset is infinite: their pairs have no r^2 and
    add nothing, to any of the other bodies' sums or counts either."""
    from paper_1912_04197_amd import api, ics

    s = ics.uniform_ball(n, seed=n + 2)
    up = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    far = [n // 3, n - 1]
    pos, mass = s.pos.copy(), s.mass.copy()
    pos[far] = [[1e308, 0.0, 0.0], [-1e308, 0.0, 0.0]]
    near = np.setdiff1d(np.arange(n), far)
    ctx = api.Context(n, leaf_size=8, precision="fp64", counts=True)
    ref = ctx.compute_accel_direct(up(pos[near]), up(mass[near]), softening=1e-2).cpu().numpy()
    scale = 1e-12 * np.linalg.norm(ref, axis=1).max()
    got = [ctx.compute_accel_direct(up(pos), up(mass), softening=1e-2),
           ctx.compute_accel(up(pos), up(mass), 0.5, softening=1e-2)]
    counts = ctx.walk_counts(n).cpu().numpy()
    for acc in (t.cpu().numpy() for t in got):
        assert np.all(acc[far] == 0.0)
        assert np.abs(acc[near] - ref).max() <= scale
    assert np.all(counts == [0, n - 1])  # one leaf: no cell is smaller than the box


@pytest.mark.parametrize("per_body", [False, True])
def test_extreme_masses_in_every_kind_of_build(per_body):
    """Walks of scenes with a mass out of the plain range: several steps in a call equal
    single-step calls bit for bit (the state keeps what the first build found), and
    every scene of a batch equals its own call."""
    from paper_1912_04197_amd import api, ics

    up = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    s = ics.rubble_pile(6000, seed=3)
    s.mass[77] = 1e-150
    eps = up(s.eps) if per_body else None
    ctx = api.Context(s.n, leaf_size=8, precision="fp64")
    runs = []
    for steps in (3, 1):
        p, v, m = up(s.pos), up(s.vel), up(s.mass)
        a = ctx.compute_accel(p, m, 0.5, softening=1e-3, eps=eps)
        for _ in range(3 // steps):
            ctx.step_leapfrog(p, v, m, a, 1e-3, steps, theta=0.5, softening=1e-3, eps=eps)
        runs.append((p, v, a))
    assert all(torch.equal(x, y) for x, y in zip(*runs))
    sizes = (300, 6000, 40)
    off = np.concatenate([[0], np.cumsum(sizes)])
    parts = [ics.uniform_ball(k, seed=k) for k in sizes]
    parts[0].mass[5] = 1e-150
    pos, mass = (up(np.concatenate([getattr(q, a) for q in parts])) for a in ("pos", "mass"))
    many = api.Context(sum(sizes), leaf_size=8, precision="fp64", max_scenes=3, walk_group=16)
    got = many.batched_accel(off, pos, mass, 0.5, softening=1e-3)
    one = api.Context(6000, leaf_size=8, precision="fp64", walk_group=16)
    for k in range(3):
        sl = slice(int(off[k]), int(off[k + 1]))
        want = one.compute_accel(pos[sl], mass[sl], 0.5, softening=1e-3)
        assert torch.equal(got[sl], want)
