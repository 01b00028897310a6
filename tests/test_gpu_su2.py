"""GPU parity of the SU(2) x U(1) doublet path (Sec. 6) against the FP64 oracle."""
import math

import numpy as np
import pytest

import oracle
from paper_2006_15122_amd import synth
from test_gpu_scalar import check_shells

pytestmark = pytest.mark.gpu

KEYS = ("a", "b", "EK", "EG", "EV", "EK_A", "EG_A", "EK_B", "EG_B", "EV_quartic")
STATE = ("phi", "pi", "links", "su2", "piA", "piB")


def _lattice(cfg):
    from paper_2006_15122_amd.lattice import Lattice

    return Lattice(cfg, device="cuda:0")


def _cfg(N, precision="fp32", **kw):
    c = dict(synth.config_su2u1(N=N), precision=precision)
    c.update(kw)
    return c


def _set(lat, st):
    lat.set_state(st["phi"], st["pi"], st["a"], st["b"], links=st["links"], su2=st["su2"], piA=st["piA"],
                  piB=st["piB"])


def compare(g, o, tol, what):
    bad = {}
    for k in KEYS:
        if o[k] == 0.0:
            continue
        r = abs(g[k] - o[k]) / abs(o[k])
        if not r <= tol:
            bad[k] = r
    sc = math.sqrt(o["meansq"])
    for c in range(4):
        r = abs(g["mean"][c] - o["mean"][c]) / sc
        if not r <= tol:
            bad[f"mean{c}"] = r
    r = abs(g["meansq"] - o["meansq"]) / o["meansq"]
    if not r <= tol:
        bad["meansq"] = r
    assert not bad, (what, bad)
    return max([abs(g[k] - o[k]) / abs(o[k]) for k in KEYS if o[k] != 0.0])


@pytest.mark.parametrize("N", [32, 64])
def test_su2_device_initial_state_matches_oracle_fp64(N):
    cfg = _cfg(N, "fp64")
    lat = _lattice(cfg)
    st = oracle.su2_vacuum_ic(cfg)
    s = lat.get_state()
    for key in STATE:
        ref = st[key]
        assert np.max(np.abs(s[key] - ref)) < 1e-12 * max(np.max(np.abs(ref)), 1e-30), key
    assert abs(s["b"] - st["b"]) < 1e-12 * st["b"]
    e = lat.energies()
    assert e["gauss"] < 1e-12 and e["gauss_B"] < 1e-12
    compare(e, oracle.su2_sync_observe(oracle.su2_model(cfg), st), 1e-12, "initial state")


@pytest.mark.parametrize("integ,nsteps", [("lf2", 100), ("vv2", 60), ("vv4", 20)])
def test_su2_fp64_parity_and_both_gauss_laws(integ, nsteps):
    # couplings e = g = 0.5: at the workload's e = 0.1 the U(1) plaquette angles stay
    # near 1e-4, where the oracle's own 1 - Re V_ij (links kept as (Re, Im), unit only
    # to rounding) carries ~1e-16 per plaquette against Phi^2/2 ~ 5e-9, a 1e-10
    # relative floor in E_G^A on its side; the GPU keeps the phases
    cfg = _cfg(32, "fp64", integrator=integ, e=0.5, g=0.5)
    st = oracle.su2_vacuum_ic(cfg)
    m = oracle.su2_model(cfg)
    lat = _lattice(cfg)
    _set(lat, st)
    h = cfg["dt"]
    if integ == "lf2":
        oracle.su2_lf_startup(m, st, h)
    half = nsteps // 2
    for k in range(2):
        lat.step(half)
        if integ == "lf2":
            oracle.su2_lf_steps(m, st, h, half, omp=True)
            o = oracle.su2_lf_observe(m, st, h)
        else:
            oracle.su2_vv_steps(m, st, h, integ, half, omp=True)
            o = oracle.su2_sync_observe(m, st)
        g = lat.energies()
        compare(g, o, 1e-10, f"{integ} fp64 step {half * (k + 1)}")
        assert g["gauss"] < 1e-12 and g["gauss_B"] < 1e-12, (g["gauss"], g["gauss_B"])
    assert o["EG_B"] > 0.0 and o["EG_A"] > 0.0
    s = lat.get_state()
    assert s["staggered"] == (integ == "lf2") and s["step"] == nsteps
    for key in STATE:
        assert np.max(np.abs(s[key] - st[key])) < 1e-10 * np.max(np.abs(st[key])), key


@pytest.mark.parametrize("integ,nsteps", [("vv2", 200), ("lf2", 200)])
def test_su2_fp32_parity_64(integ, nsteps):
    cfg = _cfg(64, "fp32", integrator=integ)
    st = oracle.su2_vacuum_ic(cfg)
    m = oracle.su2_model(cfg)
    lat = _lattice(cfg)
    _set(lat, st)
    h = cfg["dt"]
    if integ == "lf2":
        oracle.su2_lf_startup(m, st, h)
    for k in range(4):
        lat.step(nsteps // 4)
        if integ == "lf2":
            oracle.su2_lf_steps(m, st, h, nsteps // 4, omp=True)
            o = oracle.su2_lf_observe(m, st, h)
        else:
            oracle.su2_vv_steps(m, st, h, integ, nsteps // 4, omp=True)
            o = oracle.su2_sync_observe(m, st)
        g = lat.energies()
        w = compare(g, o, 1e-5, f"{integ} fp32 step {nsteps // 4 * (k + 1)}")
        print(integ, "step", nsteps // 4 * (k + 1), "worst %.2e gauss %.2e gauss_B %.2e" % (w, g["gauss"], g["gauss_B"]),
              flush=True)
        assert g["gauss"] < 1e-5 and g["gauss_B"] < 1e-5, (g["gauss"], g["gauss_B"])
    s = lat.get_state()
    assert np.max(np.abs((s["su2"] ** 2).sum(axis=1) - 1.0)) < 1e-6


def test_su2_doublet_spectra_match_oracle():
    from paper_2006_15122_amd.lattice import SPEC_U1_PHI, SPEC_U1_PI

    for precision, tol in (("fp64", 1e-10), ("fp32", 1e-5)):
        cfg = _cfg(64, precision)
        lat = _lattice(cfg)
        lat.step(40)
        s = lat.get_state()
        for which, key in ((SPEC_U1_PHI, "phi"), (SPEC_U1_PI, "pi")):
            g = lat.spectrum(which)
            parts = [oracle.spectrum(s[key][c], cfg["kIR"]) for c in range(4)]
            o = dict(parts[0])
            o["S"] = sum(p["S"] for p in parts)
            N, dx = 64, oracle.lattice_dx(64, cfg["kIR"])
            bb = np.arange(len(o["S"]), dtype=np.float64)
            o["delta"] = np.zeros(len(o["S"]))
            o["delta"][1:] = (cfg["kIR"] * bb[1:]) ** 3 * (dx / N) ** 3 / (2 * math.pi ** 2) * o["S"][1:] / (
                4 * math.pi * bb[1:] ** 2)
            check_shells(g, o, tol, f"su2 {precision} {key}")
        # a single real component
        g = lat.spectrum(2)
        check_shells(g, oracle.spectrum(s["phi"][2], cfg["kIR"]), tol, f"su2 {precision} component 2")


def test_su2_full_size_128_fp32_against_oracle():
    # the benchmarked workload at its full size: 10 steps against the live oracle
    cfg = _cfg(128, "fp32")
    st = oracle.su2_vacuum_ic(cfg)
    m = oracle.su2_model(cfg)
    lat = _lattice(cfg)
    _set(lat, st)
    lat.step(10)
    oracle.su2_vv_steps(m, st, cfg["dt"], "vv2", 10, omp=True)
    o = oracle.su2_sync_observe(m, st)
    g = lat.energies()
    print("128^3 worst %.2e gauss %.2e gauss_B %.2e" % (compare(g, o, 1e-5, "128^3"), g["gauss"], g["gauss_B"]))
    assert g["gauss"] < 1e-5 and g["gauss_B"] < 1e-5


def test_su2_energy_constraint_ladder_and_orders():
    """The accuracy tests of the SU(2) x U(1) simulations (Sec. 8.3.1): the
    Friedmann-constraint violation Delta_e falls with the integrator's order
    (VV4 about twentyfold below VV2 there), and both Gauss laws hold to
    round-off whatever the integrator.  Each integrator's order is measured:
    halving the step from 0.005 to 0.0025 divides Delta_e at eta = 10 by 2^p
    (p = 2 for the staggered leapfrog and VV2, up to 10 for VV10) within a
    factor 1.5.  The doublet at 32^3 in FP64 storage with e = g = 0.5."""
    from paper_2006_15122_amd.lattice import Lattice

    eta = 10.0
    hc = {}
    for dt in (0.005, 0.0025):
        for integ in ("lf2", "vv2", "vv4", "vv6", "vv8", "vv10"):
            cfg = _cfg(32, "fp64", integrator=integ, dt=dt, e=0.5, g=0.5)
            lat = Lattice(cfg, device="cuda:0")
            lat.step(int(round(eta / dt)))
            e = lat.energies()
            lat.close()
            hc[dt, integ] = e["hc"]
            print(f"dt {dt} {integ}: Delta_e {e['hc']:.3e} gauss {e['gauss']:.1e} {e['gauss_B']:.1e}", flush=True)
            assert e["gauss"] < 1e-12 and e["gauss_B"] < 1e-12, (dt, integ, e["gauss"], e["gauss_B"])
    for integ, p in (("lf2", 2), ("vv2", 2), ("vv4", 4), ("vv6", 6), ("vv8", 8), ("vv10", 10)):
        r = hc[0.005, integ] / hc[0.0025, integ]
        assert 2.0 ** p / 1.5 < r < 2.0 ** p * 1.5, (integ, p, r)
    order = ("vv2", "vv4", "vv6", "vv8", "vv10")
    for lo, hi in zip(order, order[1:]):
        assert hc[0.0025, hi] <= max(hc[0.0025, lo] / 10.0, 1e-12), (lo, hi)
    assert 0.5 < hc[0.0025, "lf2"] / hc[0.0025, "vv2"] < 4.0


@pytest.mark.parametrize("precision,N,integ,nsteps,tol", [
    ("fp64", 32, "lf2", 3, 1e-11), ("fp64", 64, "vv4", 1, 1e-11), ("fp32", 32, "vv2", 3, 2e-5),
    ("fp32", 96, "lf2", 2, 2e-5), ("fp32", 64, "vv4", 1, 2e-5)])
def test_su2_pass_sites_on_a_rough_state(precision, N, integ, nsteps, tol):
    """Site by site against the oracle on a state that is rough at the scale of
    a site (phases over the whole circle, links all over SU(2)), at the sizes
    where a block marches one plane and several; every component, tile edges
    and periodic seams included.  FP32: single sites, a few hundred roundings
    of 6e-8 each; FP64 the same with 1e-16."""
    rng = np.random.default_rng(17)
    cfg = _cfg(N, precision, integrator=integ, e=0.5, g=0.5)
    st = oracle.su2_vacuum_ic(cfg)
    th = rng.uniform(-math.pi, math.pi, (3, N, N, N)).astype(np.float32).astype(np.float64)
    u = rng.normal(size=(3, 4, N, N, N))
    u = (u / np.sqrt((u ** 2).sum(1, keepdims=True))).astype(np.float32).astype(np.float64)
    u /= np.sqrt((u ** 2).sum(1, keepdims=True))
    st["links"] = np.stack([np.cos(th), np.sin(th)], axis=1)
    st["su2"] = u
    for key, amp in (("phi", 0.5), ("pi", 0.5), ("piA", 5.0), ("piB", 5.0)):
        st[key] = amp * rng.normal(size=st[key].shape).astype(np.float32).astype(np.float64)
    m = oracle.su2_model(cfg)
    lat = _lattice(cfg)
    _set(lat, st)
    h = cfg["dt"]
    before = lat.spectrum(0)
    lat.step(nsteps)
    if integ == "lf2":
        oracle.su2_lf_startup(m, st, h)
        oracle.su2_lf_steps(m, st, h, nsteps, omp=True)
    else:
        oracle.su2_vv_steps(m, st, h, integ, nsteps, omp=True)
    s = lat.get_state()
    for key in STATE:
        scale = np.sqrt(np.mean(st[key] ** 2))
        assert np.max(np.abs(s[key] - st[key])) < tol * max(scale, np.max(np.abs(st[key])) / 10), key
    assert abs(s["a"] - st["a"]) < tol * st["a"] and abs(s["b"] - st["b"]) < tol * abs(st["b"])
    # the chain's records stay in their regions: the shell geometry behind them is untouched
    after = lat.spectrum(0)
    assert np.array_equal(before["k"], after["k"]) and np.array_equal(before["count"], after["count"])


def _scale_factor_force(cfg, e):
    """b' = K_a at the energies e (Sec. 5.4.1 and Sec. 6.3.1)."""
    al, a = cfg["alpha"], e["a"]
    gauge = e["EK_A"] + e["EG_A"] + e["EK_B"] + e["EG_B"]
    return cfg["fstar_over_mp"] ** 2 / 3.0 * a ** (1.0 + 2.0 * al) * (
        (al - 2.0) * e["EK"] + al * e["EG"] + (al + 1.0) * e["EV"] + (al - 1.0) * gauge)


@pytest.mark.parametrize("integ", ["lf2", "vv2"])
@pytest.mark.parametrize("seed", [1, 2, 3])
def test_su2_step_sums_carry_the_bits_of_the_observation_sums(integ, seed):
    """b moves by the force of the energies that an observation of the same
    state reports: both add the same FP32 terms of a site to FP64 sums one by
    one.  The state is the same at every site, so that a rounding of two terms
    added in FP32 (up to 6e-8 of them) is the same everywhere and does not
    average out.  The sums differ by the order of 32^3 FP64 additions of equal
    sign (at most 4e-12 of b's change); each b carries 1e-16 of itself."""
    rng = np.random.default_rng(seed)
    N = 32
    cfg = _cfg(N, "fp32", integrator=integ, alpha=0.0, m2=(1.0, 0.0), e=0.5, g=0.5, omega_over_f=1.0,
               fstar_over_mp=1.0)
    st = oracle.su2_vacuum_ic(cfg)
    one = np.ones((N, N, N))
    const = lambda shape: rng.uniform(0.3, 1.0, shape).astype(np.float32).astype(np.float64)[..., None, None, None] * one
    st["phi"], st["pi"] = const(4), const(4)
    st["piA"], st["piB"] = const(st["piA"].shape[:-3]), const(st["piB"].shape[:-3])
    st["links"] = np.stack([np.ones((3, N, N, N)), np.zeros((3, N, N, N))], axis=1)
    st["su2"] = np.stack([one * (k == 0) for k in range(4)])[None].repeat(3, axis=0)
    h = cfg["dt"]
    lat, ahead = _lattice(cfg), _lattice(cfg)
    for x in (lat, ahead):
        _set(x, st)

    def b_of(x):
        return x.get_state()["b"]

    def close(b, before, terms, what):
        want = sum(terms)
        got = b - before
        assert abs(got - want) < 1e-11 * sum(map(abs, terms)) + 1e-15 * abs(b), (what, got, want, got / want - 1.0)

    b0, f0 = b_of(lat), _scale_factor_force(cfg, lat.energies())
    if integ == "lf2":
        lat.step(0)
        ahead.step(0)
        b1, f1 = b_of(lat), _scale_factor_force(cfg, lat.energies())
        close(b1, b0, [-0.5 * h * f0], "start-up kick")
        ahead.step(1)
        close(b_of(ahead), b1, [h * f1], "kick")
        f2 = _scale_factor_force(cfg, ahead.energies())
        lat.step(2)
        close(b_of(lat), b1, [h * f1, h * f2], "kick and drift with kick")
    else:
        ahead.step(1)
        f1 = _scale_factor_force(cfg, ahead.energies())
        close(b_of(ahead), b0, [0.5 * h * f0, 0.5 * h * f1], "one step")
        # (the closing state's energies are lat's own: its merged kick rounds the
        # momenta once where two single steps round them twice)
        lat.step(2)
        f2 = _scale_factor_force(cfg, lat.energies())
        close(b_of(lat), b0, [0.5 * h * f0, h * f1, 0.5 * h * f2], "two steps")


@pytest.mark.parametrize("precision,N", [("fp32", 32), ("fp64", 32)])
def test_su2_pass_without_drift_takes_stored_phases_as_they_are(precision, N):
    """U(1) phases of many turns, written through the component pointers: the
    observation and the start-up kick take the sine of the stored phase, and
    the kick leaves it as it is."""
    from test_gpu_u1 import phases_over_many_turns, run_phases_over_many_turns

    rng = np.random.default_rng(6)
    cfg = _cfg(N, precision, integrator="lf2", e=0.5, g=0.5)
    st = oracle.su2_vacuum_ic(cfg)
    for key in ("phi", "pi", "piA", "piB"):
        st[key] = 0.5 * rng.normal(size=st[key].shape)
    th = phases_over_many_turns(N, rng)
    lat = _lattice(cfg)
    _set(lat, st)
    for key in ("phi", "pi", "piA", "piB"):
        st[key] = lat.get_state()[key]
    st["links"] = np.ascontiguousarray(np.stack([np.cos(th), np.sin(th)], axis=1))
    run_phases_over_many_turns(lat, 8, th, lambda: oracle.su2_sync_observe(oracle.su2_model(cfg), st))


def test_su2_stored_phases_past_counting():
    from test_gpu_u1 import run_phases_past_counting

    cfg = _cfg(32, "fp32", integrator="lf2", e=0.5, g=0.5)
    lat = _lattice(cfg)
    _set(lat, oracle.su2_vacuum_ic(cfg))
    run_phases_past_counting(lat, 8)
