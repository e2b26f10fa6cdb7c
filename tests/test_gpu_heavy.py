"""Heavy home leaves: isolated sets of whole leaves (above 24,576 particles at leaf
size 16) leave the home leaves that see hundreds of others to a second launch, with a
wave for each of their particles.

Here with unequal masses, the quintic kernel, artificial conductivity and
per-particle viscosity (against the oracle), beside sets without heavy leaves in a
batch, in sub-steps and in captured steps (bits of the single and the eager calls).

Tolerances against the oracle: those of test_gpu_parity (FP64 1e-10 relative, a and
du/dt of the per-particle scale, counts exact; FP32-pair 1e-5, Omega 1e-4, a and du/dt
1e-4 of the scale).
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_1709_04488_amd import workloads as W  # noqa: E402
from test_gpu_paths import cluster_with_outliers  # noqa: E402

KEYS = ("h", "rho", "omega", "nngb", "ax", "ay", "az", "dudt", "vsig", "dt", "nforce")


@pytest.fixture(scope="module")
def sph():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1709_04488_amd import sph as s
    s.load()
    return s


def _set(n=24600, equal_m=True, seed=67):
    w = cluster_with_outliers(n_cluster=n, seed=seed)
    a = dict(w.arrays)
    if not equal_m:
        f = np.random.default_rng(seed + 1).uniform(0.5, 1.5, a["m"].size)
        a["m"], a["h"] = a["m"] * f, a["h"] * np.cbrt(f)
    return a, w.setup


@pytest.mark.parametrize("precision", [0, 1])
def test_every_heavy_particle_has_a_wave(sph, precision):
    """Guesses four times too large make every leaf heavy: the walks of the first
    launch and one per particle in the second.  The results are those of near guesses."""
    n = 26000
    w = W.plummer(n, seed=3)
    print(f"case: all leaves heavy precision={precision}", flush=True)
    out = {}
    for factor in (1.0, 4.0):
        with sph.Context(sph.Params.from_setup(w.setup, precision=precision)) as ctx:
            p = sph.Particles.from_host({**w.arrays, "h": factor * w.arrays["h"]})
            ctx.evaluate(p)
            ctx.sync()
            walks = ctx.state_info()["dens_walks"]
            assert walks > n if factor == 4.0 else walks < n
            out[factor] = p.host(*KEYS)
    tol = 1e-10 if precision == 0 else 1e-5
    for k in ("h", "rho", "vsig", "dt"):
        assert np.max(np.abs(out[4.0][k] / out[1.0][k] - 1.0)) < tol, k
    if precision == 0:
        for k in ("nngb", "nforce"):
            assert np.array_equal(out[4.0][k], out[1.0][k]), k


@pytest.mark.parametrize("precision,kernel,equal_m,over", [
    (0, 1, False, {}), (0, 0, False, {"alpha_ac": 1.0}), (1, 0, False, {}), (1, 1, True, {"alpha_ac": 1.0}),
    (0, 0, True, {"alpha": "per particle"})])
def test_heavy_leaves_match_oracle(sph, orc, precision, kernel, equal_m, over):
    a, setup = _set(equal_m=equal_m)
    setup = {**setup, "kernel": kernel}
    if "alpha" in over:
        a["alpha"] = np.random.default_rng(5).uniform(0.1, 1.0, a["m"].size)
    else:
        setup.update(over)
    print(f"case: heavy leaves precision={precision} kernel={kernel} equal_m={equal_m} {over}", flush=True)
    ref = orc.evaluate(orc.Params(**setup), a["x"], a["y"], a["z"], a["vx"], a["vy"], a["vz"], a["m"], a["u"],
                       a["h"], alpha=a.get("alpha"))
    assert np.all(ref["nngb"][-5:] >= 0.9 * a["m"].size)   # (the case is what it is meant to be)
    with sph.Context(sph.Params.from_setup(setup, precision=precision)) as ctx:
        p = sph.Particles.from_host(a)
        ctx.evaluate(p)
        ctx.sync()
        out = p.host(*KEYS)
    tol, atol = ((1e-10, 1e-10), (1e-5, 1e-4))[precision]
    for k in ("h", "rho", "omega", "vsig", "dt"):
        assert np.max(np.abs(out[k] / ref[k] - 1.0)) < (1e-4 if k == "omega" and precision else tol), k
    for k, sk in (("ax", "scale_a"), ("ay", "scale_a"), ("az", "scale_a"), ("dudt", "scale_u")):
        assert np.max(np.abs(out[k] - ref[k]) / ref[sk]) < atol, k
    if precision == 0:
        for k in ("nngb", "nforce"):
            assert np.array_equal(out[k], ref[k]), k


@pytest.mark.parametrize("precision", [0, 1])
def test_heavy_leaves_in_a_batch(sph, precision):
    """Beside a small isolated set, a periodic one and a large one without heavy
    leaves: the bits of each alone."""
    plummer = W.plummer(3000, seed=8)
    lattice = W.jittered_lattice(20, seed=9)
    rng = np.random.default_rng(10)
    even = dict(W.plummer(26000, seed=11).arrays)
    even.update({k: rng.uniform(0, 1, 26000) for k in "xyz"})
    even["h"] = np.full(26000, 1.2 * 26000 ** (-1.0 / 3.0))
    sets = [(plummer.arrays, plummer.setup), _set(), (lattice.arrays, lattice.setup), (even, plummer.setup),
            _set(25000, False, 71)]
    print(f"case: heavy leaves in a batch precision={precision}", flush=True)
    params = [sph.Params.from_setup(s, precision=precision) for _, s in sets]
    alone = []
    for (a, _), q in zip(sets, params):
        with sph.Context(q) as ctx:
            p = sph.Particles.from_host(a)
            ctx.evaluate(p)
            ctx.sync()
            alone.append(p.host(*KEYS))
    for order in (range(5), (1, 4, 0, 3, 2)):   # (the claims go through the first set's counters)
        ctxs = [sph.Context(params[i]) for i in order]
        parts = [sph.Particles.from_host(sets[i][0]) for i in order]
        sph.batch_evaluate(ctxs, parts)
        for c in ctxs:
            c.sync()
        for i, p in zip(order, parts):
            out = p.host(*KEYS)
            for k in KEYS:
                assert np.array_equal(out[k], alone[i][k]), (i, k)
        for c in ctxs:
            c.close()


def _state(sph, ctx, a, level=False):
    q = sph.Particles.from_host(a)
    if level:
        q.with_level()
    ctx.download_state(q)
    ctx.sync()
    return q.host()


STATE = ("x", "y", "z", "vx", "vy", "vz", "u", "h", "rho", "ax", "ay", "az", "dudt", "nngb", "nforce")


def test_heavy_leaves_in_captured_steps(sph):
    a, setup = _set()
    print("case: heavy leaves in captured steps", flush=True)
    stream = torch.cuda.Stream()
    params = sph.Params.from_setup(setup)
    eager, graph = sph.Context(params, stream=stream), sph.Context(params, stream=stream)
    with torch.cuda.stream(stream):
        pe, pg = sph.Particles.from_host(a), sph.Particles.from_host(a)
        eager.upload_state(pe)
        graph.upload_state(pg)
        graph.capture_steps(0.0)
        for rep in range(3):
            eager.step(0.0)
            eager.step(0.0)
            graph.replay_steps()
            stream.synchronize()
            x, y = _state(sph, eager, a), _state(sph, graph, a)
            for k in STATE:
                assert np.array_equal(x[k], y[k]), (rep, k)
    eager.close()
    graph.close()


def test_heavy_leaves_in_substeps(sph):
    """The far particles are cold and the cluster hot, so most sub-steps leave the
    heavy leaves out and some have them active: batched sub-steps give the bits of
    single ones, and other leaf sizes the same levels and, to rounding, the state."""
    a, setup = _set()
    a["u"] = a["u"].copy()
    a["u"][:100] *= 300.0
    setup = {**setup, "block_lmax": 16}
    print("case: heavy leaves in sub-steps", flush=True)

    def run(leaf, with_other):
        params = sph.Params.from_setup(setup, leaf_size=leaf)
        ctxs = [sph.Context(params)]
        sets = [a]
        if with_other:
            ctxs.insert(0, sph.Context(params))
            sets.insert(0, _set(24700, True, 77)[0])
        for c, s in zip(ctxs, sets):
            c.upload_state(sph.Particles.from_host(s))
        seen = set()
        for _ in range(12):
            sph.batch_substep(ctxs) if with_other else ctxs[0].substep()
            seen.add(ctxs[-1].state_info()["block_active"])
        for c in ctxs:
            c.sync()
        out = _state(sph, ctxs[-1], a, level=True)
        for c in ctxs:
            c.close()
        return out, seen

    single, seen = run(16, False)
    assert len(seen) > 1
    batched, _ = run(16, True)
    for k in STATE + ("level",):
        assert np.array_equal(single[k], batched[k]), k
    other, _ = run(32, False)
    assert np.array_equal(single["level"], other["level"])
    for k in ("x", "y", "z", "u", "h", "rho"):
        assert np.max(np.abs(single[k] - other[k])) < 1e-9 * np.max(np.abs(single[k])), k
