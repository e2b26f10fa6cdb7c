"""Sets at the edges of what the entry points take: any unit of length, values
that are not finite, leaves that are wide against their particles' reaches.

A set in another unit of length is the same set: with a power of two between the
units every FP64 operation rounds alike, so the results have to scale to the bit
(h with the unit, rho with its cube, Omega, counts and the signal speed not at all,
the accelerations with its inverse).
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_1709_04488_amd import workloads as W  # noqa: E402


@pytest.fixture(scope="module")
def sph():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1709_04488_amd import sph as s
    s.load()
    return s


def _set(n, periodic, equal_m=True, seed=3):
    rng = np.random.default_rng(seed)
    if periodic:
        a = {k: rng.uniform(0, 1, n) for k in "xyz"}
        a["h"] = 1.2 * n ** (-1.0 / 3.0) * rng.uniform(0.8, 1.2, n)
    else:
        w = W.plummer(n, seed)
        a = {k: w.arrays[k].copy() for k in ("x", "y", "z", "h")}
    a.update({k: rng.normal(0, 0.3, n) for k in ("vx", "vy", "vz")})
    a["m"] = np.full(n, 1.0 / n) if equal_m else rng.uniform(0.5, 1.5, n) / n
    a["u"] = rng.uniform(0.3, 2.0, n)
    return a, W.default_setup(periodic=periodic)


def _in_unit(a, setup, unit):
    """The set with lengths in units of 1 / unit."""
    a = {k: v * unit if k in ("x", "y", "z", "h") else v for k, v in a.items()}
    return a, dict(setup, lo=tuple(unit * v for v in setup["lo"]), hi=tuple(unit * v for v in setup["hi"]))


def _run(sph, a, setup, forces=True, **kw):
    """(outputs, status) of one evaluation, or of the density alone."""
    with sph.Context(sph.Params.from_setup(setup, **kw)) as ctx:
        p = sph.Particles.from_host(a)
        ctx.evaluate(p) if forces else ctx.density(p)
        status = ctx.sync_status()
        return p.host(), status


# powers of the unit in each output
UNIT = {"h": 1, "rho": -3, "omega": 0, "vsig": 0, "dt": 1, "ax": -1, "ay": -1, "az": -1, "dudt": -1}


@pytest.mark.parametrize("kernel", [0, 1])
@pytest.mark.parametrize("periodic,leaf", [(True, 16), (False, 8), (False, 32)])
@pytest.mark.parametrize("log2_unit", [-110, -66, 64, 83])
def test_fp64_in_any_unit(sph, log2_unit, periodic, leaf, kernel):
    a, setup = _set(3000, periodic)
    print(f"case: unit 2^{log2_unit} periodic={periodic} leaf={leaf} kernel={kernel}", flush=True)
    ref, ok = _run(sph, a, setup, leaf_size=leaf, kernel=kernel)
    unit = 2.0 ** log2_unit
    out, status = _run(sph, *_in_unit(a, setup, unit), leaf_size=leaf, kernel=kernel)
    assert status == ok
    for k in ("nngb", "nforce"):
        assert np.array_equal(out[k], ref[k]), k
    for k, power in UNIT.items():
        assert np.array_equal(out[k], ref[k] * unit ** power), k


@pytest.mark.parametrize("equal_m", [True, False])
@pytest.mark.parametrize("periodic,kernel", [(True, 0), (False, 1)])
@pytest.mark.parametrize("log2_unit", [-50, 55, 60])
def test_fp32_density_in_any_unit(sph, log2_unit, periodic, kernel, equal_m):
    """Up to where squares of lengths leave the single-precision range (the force
    loop's h^-4 leaves it earlier)."""
    a, setup = _set(3000, periodic, equal_m)
    print(f"case: fp32 unit 2^{log2_unit} periodic={periodic} kernel={kernel} equal_m={equal_m}", flush=True)
    ref, ok = _run(sph, a, setup, forces=False, kernel=kernel, precision=1)
    unit = 2.0 ** log2_unit
    out, status = _run(sph, *_in_unit(a, setup, unit), forces=False, kernel=kernel, precision=1)
    assert status == ok
    assert np.array_equal(out["nngb"], ref["nngb"])
    for k in ("h", "rho", "omega"):
        assert np.array_equal(out[k], ref[k] * unit ** UNIT[k]), k


def _without(a, i):
    return {k: np.delete(v, i) for k, v in a.items()}


def _same_but(out, ref, i, precision):
    """The other particles' results as in the set without particle i, to the
    tolerances of the small-set tests (another leaf structure)."""
    tol = 1e-10 if precision == 0 else 1e-4
    for k in ("nngb", "nforce"):
        d = np.delete(out[k], i) != ref[k]
        # (single precision: a pair at the kernel's edge may fall to either side)
        assert np.count_nonzero(d) <= (0 if precision == 0 else 5), k
    for k in ("h", "rho", "omega", "vsig", "dt", "ax", "ay", "az", "dudt"):
        o = np.delete(out[k], i)
        scale = np.abs(ref[k]) if k in ("h", "rho", "omega", "vsig", "dt") else np.abs(ref[k]).max()
        assert np.max(np.abs(o - ref[k]) / scale) < tol, k


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("periodic,kernel,n", [(True, 0, 700), (True, 1, 2000), (False, 0, 2000)])
def test_nan_position_stays_alone(sph, precision, periodic, kernel, n):
    """A particle whose position is not a number is flagged and is nobody's
    neighbour (the small periodic sets list every candidate: their leaves see the
    box's images ambiguously)."""
    a, setup = _set(n, periodic)
    i = 555
    a["x"][i] = np.nan
    print(f"case: nan position precision={precision} periodic={periodic} kernel={kernel} n={n}", flush=True)
    out, status = _run(sph, a, setup, kernel=kernel, precision=precision)
    assert status == sph.SPH_ENONFINITE
    ref, status = _run(sph, _without(a, i), setup, kernel=kernel, precision=precision)
    assert status == sph.SPH_OK
    _same_but(out, ref, i, precision)


@pytest.mark.parametrize("periodic,kernel", [(True, 0), (True, 1), (False, 0), (False, 1)])
def test_infinite_position_stays_alone(sph, periodic, kernel):
    """The particles that share its leaf keep their neighbours (FP64: in the
    FP32-pair mode their offsets from the leaf's centre are not finite)."""
    a, setup = _set(2000, periodic)
    i = 777
    a["x"][i] = np.inf
    print(f"case: infinite position periodic={periodic} kernel={kernel}", flush=True)
    out, status = _run(sph, a, setup, kernel=kernel)
    assert status == sph.SPH_ENONFINITE
    if not periodic:   # (the box of the keys is infinite: every particle has the same key)
        assert np.isfinite(np.delete(out["ax"], i)).all()
    ref, status = _run(sph, _without(a, i), setup, kernel=kernel)
    assert status == sph.SPH_OK
    _same_but(out, ref, i, 0)


@pytest.mark.parametrize("leaf,kernel", [(8, 0), (16, 0), (16, 1), (32, 0)])
def test_leaves_wide_against_their_reaches(sph, orc, leaf, kernel):
    """Two tight groups 1e5 smoothing lengths apart whose particles take turns in the
    input, and one far particle: the groups share the finest key cell, so leaves
    hold particles of both, and home coordinates exceed the halves' range."""
    n = 600
    rng = np.random.default_rng(13)
    pos = (np.arange(n) % 2)[:, None] * np.array([[1e-4, 0, 0]]) + rng.normal(0, 1e-9, (n, 3))
    pos[-1] = 1.0
    a = {k: pos[:, i].copy() for i, k in enumerate("xyz")}
    a.update({k: rng.normal(0, 0.3, n) for k in ("vx", "vy", "vz")})
    a["m"] = np.full(n, 1.0 / n)
    a["u"] = rng.uniform(0.3, 2.0, n)
    a["h"] = np.where(np.arange(n) == n - 1, 0.5, 4e-10)
    setup = W.default_setup(periodic=False)
    print(f"case: wide leaves leaf={leaf} kernel={kernel}", flush=True)
    ref = orc.evaluate(orc.Params(**{**setup, "kernel": kernel}), a["x"], a["y"], a["z"], a["vx"], a["vy"], a["vz"],
                       a["m"], a["u"], a["h"])
    out, status = _run(sph, a, setup, leaf_size=leaf, kernel=kernel)
    assert status == sph.SPH_OK
    for k in ("nngb", "nforce"):
        assert np.array_equal(out[k], ref[k]), k
    for k in ("h", "rho", "omega", "vsig", "dt"):
        assert np.max(np.abs(out[k] / ref[k] - 1.0)) < 1e-10, k
    for k, sk in (("ax", "scale_a"), ("ay", "scale_a"), ("az", "scale_a"), ("dudt", "scale_u")):
        assert np.max(np.abs(out[k] - ref[k]) / ref[sk]) < 1e-10, k


@pytest.mark.parametrize("precision,kernel", [(0, 0), (0, 1), (1, 0)])
@pytest.mark.parametrize("mass", [np.inf, np.nan])
def test_mass_that_is_not_finite_stays_within_reach(sph, mass, precision, kernel):
    """It spoils the particles that have it within R h, and no other's density."""
    a, setup = _set(2000, True, equal_m=False)
    i = 777
    ref, status = _run(sph, a, setup, forces=False, kernel=kernel, precision=precision)
    assert status == sph.SPH_OK
    reach = (2.0, 3.0)[kernel] * ref["h"]
    d = np.stack([a[k] - a[k][i] for k in "xyz"])
    r = np.sqrt(((d - np.round(d)) ** 2).sum(0))
    a["m"][i] = mass
    # guesses beyond the root, so that lists hold the particle for many whose
    # root does not reach it
    a["h"] = 1.1 * ref["h"]
    print(f"case: mass {mass} precision={precision} kernel={kernel}", flush=True)
    out, status = _run(sph, a, setup, forces=False, kernel=kernel, precision=precision)
    assert status == sph.SPH_ENONFINITE
    # (a guess that reaches it gives no Newton step to go by)
    far = r > 1.1 * reach * (1.0 + 1e-6)
    assert np.count_nonzero(far & (r < 1.15 * 1.1 * reach)) > 5   # (the case is what it is meant to be)
    for k in ("h", "rho", "omega"):
        assert np.max(np.abs(out[k][far] / ref[k][far] - 1.0)) < (1e-10 if precision == 0 else 1e-5), k
    if precision == 0:
        assert np.array_equal(out["nngb"][far], ref["nngb"][far])


@pytest.mark.parametrize("precision,kernel,passes", [(0, 0, 50), (0, 0, 12), (0, 1, 50), (0, 1, 12), (1, 0, 8)])
@pytest.mark.parametrize("n", [2, 3, 4])
def test_no_root_keeps_omega(sph, n, kernel, precision, passes):
    """So few particles have no h that solves the h-rho relation: h grows until the
    passes end, Omega falls with (r / h)^2 towards zero, and the solve is reported as
    not converged, with finite results."""
    rng = np.random.default_rng(n)
    a = {k: rng.uniform(0, 1, n) for k in "xyz"}
    a.update({k: rng.normal(0, 0.3, n) for k in ("vx", "vy", "vz")})
    a["m"] = np.full(n, 1.0 / n)
    a["u"] = np.ones(n)
    a["h"] = np.full(n, 1.0)
    print(f"case: no root n={n} kernel={kernel} precision={precision} passes={passes}", flush=True)
    out, status = _run(sph, a, W.default_setup(periodic=False), kernel=kernel, precision=precision,
                       h_max_iter=passes)
    assert status == sph.SPH_ENOTCONVERGED
    for k in ("h", "rho", "omega", "ax", "ay", "az", "dudt", "vsig", "dt"):
        assert np.isfinite(out[k]).all(), k
    assert np.array_equal(out["nngb"], np.full(n, n - 1))
    pos = np.stack([a[k] for k in "xyz"])
    q = np.sqrt(((pos[:, :, None] - pos[:, None, :]) ** 2).sum(0)) / out["h"][:, None]
    if kernel:   # q f' and f, exact to (q^4) where q is small: expanded about q = 0
        f = 66.0 - 60.0 * q ** 2 + 30.0 * q ** 4
        qdf = -120.0 * q ** 2 + 120.0 * q ** 4
    else:
        f = 1.0 - 1.5 * q ** 2 + 0.75 * q ** 3
        qdf = -3.0 * q ** 2 + 2.25 * q ** 3
    omega = -qdf.sum(1) / (3.0 * f.sum(1))
    if passes < 50:   # (f' in its B-spline form rounds to some 4e-16 / q of itself: q is 1e-3 here, 1e-15 after 50)
        assert q.max() < 0.02
        assert np.max(np.abs(out["omega"] / omega - 1.0)) < (1e-3 if kernel or precision else 1e-9)


@pytest.mark.parametrize("precision,kernel", [(0, 0), (0, 1), (1, 0)])
def test_massless_particle(sph, precision, kernel):
    """h^3 rho = 0 holds for every h that reaches no other particle: h is halved from
    its guess until it does."""
    a, setup = _set(2000, True, equal_m=False)
    a["m"][[5, 900]] = 0.0
    print(f"case: massless precision={precision} kernel={kernel}", flush=True)
    out, status = _run(sph, a, setup, kernel=kernel, precision=precision)
    support = (2.0, 3.0)[kernel]
    for i in (5, 900):
        d = np.stack([a[k] - a[k][i] for k in "xyz"])
        r = np.sort(np.sqrt(((d - np.round(d)) ** 2).sum(0)))[1]
        h = a["h"][i]
        while support * h > r:
            h *= 0.5
        assert out["h"][i] == h and out["nngb"][i] == 0


@pytest.mark.parametrize("kernel", [0, 1])
def test_cold_solve_takes_few_passes(sph, kernel):
    """A cluster in a void, guesses off by up to 2: plain Newton needs up to 9 passes
    with the quintic kernel and 10 with M4, and a caller may allow no more."""
    n = 5000
    k = n * 3 // 4
    rng = np.random.default_rng(5)
    pos = np.concatenate([np.mod(rng.normal(0.5, 0.03, (k, 3)), 1), rng.uniform(0, 1, (n - k, 3))])
    a = {c: pos[:, i].copy() for i, c in enumerate("xyz")}
    a.update({c: rng.normal(0, 0.3, n) for c in ("vx", "vy", "vz")})
    a["m"] = np.full(n, 1.0 / n)
    a["u"] = rng.uniform(0.3, 2, n)
    a["h"] = np.where(np.arange(n) < k, 0.12 * k ** (-1 / 3), 1.2 * (n - k) ** (-1 / 3)) * rng.uniform(0.8, 1.2, n)
    print(f"case: passes of a cold solve kernel={kernel}", flush=True)
    out, status = _run(sph, a, W.default_setup(), kernel=kernel, h_max_iter=9 if kernel else 10)
    assert status == sph.SPH_OK


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("periodic,kernel,equal_m", [(True, 0, True), (False, 1, False)])
def test_infinite_guess_reaches_each_particle_once(sph, precision, periodic, kernel, equal_m):
    a, setup = _set(2000, periodic, equal_m)
    i = 777
    a["h"][i] = np.inf
    print(f"case: infinite guess precision={precision} periodic={periodic} kernel={kernel}", flush=True)
    out, status = _run(sph, a, setup, precision=precision, kernel=kernel)
    assert status == sph.SPH_ENONFINITE
    assert out["nngb"][i] == a["x"].size - 1 and out["nforce"][i] == a["x"].size - 1


def _uniform(n, guess=1.0, equal_m=True, seed=5):
    rng = np.random.default_rng(seed)
    a = {k: rng.uniform(0, 1, n) for k in "xyz"}
    a.update({k: rng.normal(0, 0.3, n) for k in ("vx", "vy", "vz")})
    a["m"] = np.full(n, 1.0 / n) if equal_m else rng.uniform(0.5, 1.5, n) / n
    a["u"] = rng.uniform(0.3, 2.0, n)
    a["h"] = guess * 1.2 * n ** (-1.0 / 3.0) * rng.uniform(0.9, 1.1, n)
    return a


@pytest.mark.parametrize("n,kernel,leaf", [(700, 0, 8), (700, 0, 16), (700, 0, 32), (1300, 1, 16), (2500, 0, 16)])
def test_fp32_lists_of_small_boxes(sph, orc, n, kernel, leaf):
    """Reaches that span much of the box: the images are ambiguous, and the lists
    still hold what is within reach (with equal masses up to 640 and 1,920 of them)."""
    a, setup = _uniform(n), W.default_setup()
    print(f"case: fp32 small box n={n} kernel={kernel} leaf={leaf}", flush=True)
    with sph.Context(sph.Params.from_setup(setup, precision=1, kernel=kernel, leaf_size=leaf)) as ctx:
        p = sph.Particles.from_host(a)
        ctx.evaluate(p)
        ctx.sync()
        assert ctx.state_info()["dens_list_overflows"] == 0
        out = p.host()
    ref = orc.evaluate(orc.Params(**{**setup, "kernel": kernel}), a["x"], a["y"], a["z"], a["vx"], a["vy"], a["vz"],
                       a["m"], a["u"], a["h"])
    for k in ("h", "rho", "omega", "vsig", "dt"):
        assert np.max(np.abs(out[k] / ref[k] - 1.0)) < (5e-5 if k == "omega" else 1e-5), k
    for k, sk in (("ax", "scale_a"), ("ay", "scale_a"), ("az", "scale_a"), ("dudt", "scale_u")):
        assert np.max(np.abs(out[k] - ref[k]) / ref[sk]) < 1e-4, k


@pytest.mark.parametrize("kernel,equal_m", [(0, True), (0, False), (1, True)])
def test_fp32_small_and_large_boxes_in_one_batch(sph, kernel, equal_m):
    """A set above the line of the lane-by-lane tests, with guesses that make its
    images ambiguous, gives the same bits alone and beside sets below it."""
    sets = [_uniform(700, 1.0, equal_m), _uniform(33000, 6.0, equal_m), _uniform(5000, 2.0, equal_m)]
    print(f"case: fp32 boxes in one batch kernel={kernel} equal_m={equal_m}", flush=True)
    params = sph.Params.from_setup(W.default_setup(), precision=1, kernel=kernel)
    keys = ("h", "rho", "omega", "nngb", "ax", "ay", "az", "dudt", "vsig", "nforce")
    alone = []
    for a in sets:
        with sph.Context(params) as ctx:
            p = sph.Particles.from_host(a)
            ctx.evaluate(p)
            ctx.sync()
            alone.append(p.host(*keys))
    ctxs = [sph.Context(params) for _ in sets]
    parts = [sph.Particles.from_host(a) for a in sets]
    sph.batch_evaluate(ctxs, parts)
    for c in ctxs:
        c.sync()
    for p, ref in zip(parts, alone):
        out = p.host(*keys)
        for k in keys:
            assert np.array_equal(out[k], ref[k]), (p.n, k)
    for c in ctxs:
        c.close()


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("periodic,kernel", [(True, 0), (False, 1)])
def test_undefined_guess_reaches_nothing(sph, precision, periodic, kernel):
    a, setup = _set(2000, periodic)
    i = 777
    ref, status = _run(sph, a, setup, forces=False, precision=precision, kernel=kernel)
    assert status == sph.SPH_OK
    a["h"][i] = np.nan
    print(f"case: undefined guess precision={precision} periodic={periodic} kernel={kernel}", flush=True)
    out, status = _run(sph, a, setup, forces=False, precision=precision, kernel=kernel)
    assert status == sph.SPH_ENONFINITE
    assert out["nngb"][i] <= 0 and np.isnan(out["h"][i])
    others = np.arange(2000) != i
    assert np.array_equal(out["nngb"][others], ref["nngb"][others])
    for k in ("h", "rho", "omega"):
        assert np.max(np.abs(out[k][others] / ref[k][others] - 1.0)) < (1e-10 if precision == 0 else 1e-5), k


@pytest.mark.parametrize("leaf,stages", [(8, (1, 3, 7, 16)), (16, (1, 5, 8)), (32, (1, 3, 4))])
@pytest.mark.parametrize("precision", [0, 1])
def test_density_does_not_depend_on_the_stage_depth(sph, leaf, stages, precision):
    """Also where the lists fill up (guesses of h too large, unequal masses)."""
    n = 6000
    a = _uniform(n, 2.5, equal_m=False, seed=23)
    print(f"case: stage depth leaf={leaf} precision={precision}", flush=True)
    ref, status = _run(sph, a, W.default_setup(), forces=False, leaf_size=leaf, precision=precision)
    assert status == sph.SPH_OK
    for stage in stages:
        with sph.Context(sph.Params.from_setup(W.default_setup(), leaf_size=leaf, precision=precision,
                                               stage_leaves=stage)) as ctx:
            p = sph.Particles.from_host(a)
            ctx.evaluate(p)   # (density statistics of one evaluation)
            ctx.sync()
            assert ctx.state_info()["dens_list_overflows"] > 0
            out = p.host()
        for k in ("h", "rho", "omega", "nngb"):
            assert np.array_equal(out[k], ref[k]), (stage, k)
