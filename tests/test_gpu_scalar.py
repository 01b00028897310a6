"""GPU parity of the scalar-field path (fused HIP passes) against the FP64 oracle.

Every case starts both sides from the same FP64 state (the oracle's vacuum
initial conditions, or a seeded random state) and compares the volume
observables, a, b and sampled sites.  Tolerances: 1e-10 relative for FP64
storage, 1e-5 relative for FP32 storage (FP64 sums); <phi> is compared
relative to sqrt(<phi^2>) because it oscillates through zero.
"""
import math

import numpy as np
import pytest

import oracle
from paper_2006_15122_amd import synth

pytestmark = pytest.mark.gpu

OBS_KEYS = ("a", "b", "EK", "EG", "EV", "EV_mass", "EV_quartic", "EV_int")


def _lattice(cfg):
    from paper_2006_15122_amd.lattice import Lattice

    return Lattice(cfg, device="cuda:0")


def _rel(g, o, key, scale=None):
    s = abs(o[key]) if scale is None else scale
    if s == 0.0:
        return abs(g[key])
    return abs(g[key] - o[key]) / s


def compare_obs(g, o, nf, tol, what=""):
    worst = {}
    for k in OBS_KEYS:
        if k == "EV_int" and nf < 2:
            continue
        if o[k] == 0.0 and g[k] == 0.0:
            continue
        worst[k] = _rel(g, o, k)
    for f in range(nf):
        for k in (f"EK{f}", f"EG{f}", f"meansq{f}"):
            worst[k] = _rel(g, o, k)
        worst[f"mean{f}"] = _rel(g, o, f"mean{f}", scale=math.sqrt(o[f"meansq{f}"]))
    bad = {k: v for k, v in worst.items() if not v <= tol}
    assert not bad, (what, bad)
    return max(worst.values())


def check_shells(g, o, tol, what):
    """Every shell relative to its own power.  Shells whose power is
    structurally zero (the zero mode of a field with zero mean, the
    self-conjugate corner modes the initial state leaves empty; below 1e-12
    of the largest shell) hold only transform round-off and are compared
    in absolute terms, against 1e-10 of the largest shell."""
    assert np.array_equal(g["count"], o["count"])
    top = np.max(o["S"])
    live = (o["count"] > 0) & (o["S"] > 1e-12 * top)
    rel = np.abs(g["S"][live] - o["S"][live]) / o["S"][live]
    print(what, "largest per-shell relative error %.2e over %d shells" % (rel.max(), live.sum()), flush=True)
    assert np.all(rel <= tol), (what, np.flatnonzero(live)[np.argmax(rel)], rel.max())
    assert np.all(np.abs(g["S"][~live] - o["S"][~live]) <= 1e-10 * top), what
    pos = live & (o["delta"] > 0)
    assert np.all(np.abs(g["delta"][pos] - o["delta"][pos]) <= tol * o["delta"][pos]), what


# --------------------------------------------------------------------------
# configuration 1: one scalar, 32^3, FP64, staggered leapfrog, 1000 steps
# --------------------------------------------------------------------------
def test_config1_lf2_fp64_parity_1000_steps():
    cfg = synth.config1()
    st = oracle.vacuum_ic(cfg)
    m = oracle.scalar_model(cfg)
    lat = _lattice(cfg)
    lat.set_state(st["phi"], st["pi"], st["a"], st["b"])
    phi, pi = st["phi"].copy(), st["pi"].copy()
    a, b = oracle.lf_startup(m, phi, pi, st["a"], st["b"], cfg["dt"])
    h = cfg["dt"]
    worst = 0.0
    for k in range(10):
        lat.step(100)
        a, b = oracle.lf_steps(m, phi, pi, a, b, h, 100)
        o = oracle.lf_observe(m, phi, pi, a, b, h)
        g = lat.energies()
        worst = max(worst, compare_obs(g, o, 1, 1e-10, f"step {100 * (k + 1)}"))
        assert abs(g["hc"] - o["hc"]) < 1e-10 * max(o["hc"], 1e-12) + 1e-14
    s = lat.get_state()
    assert s["staggered"] and s["step"] == 1000
    assert abs(s["eta"] - 10.0) < 1e-9
    assert np.max(np.abs(s["phi"] - phi)) < 1e-10 * np.max(np.abs(phi))
    assert np.max(np.abs(s["pi"] - pi)) < 1e-10 * np.max(np.abs(pi))
    print("config1 worst relative error", worst)


def test_config1_initial_conditions_match_oracle():
    cfg = synth.config1()
    lat = _lattice(cfg)
    st = oracle.vacuum_ic(cfg)
    s = lat.get_state()
    assert np.max(np.abs(s["phi"] - st["phi"])) < 1e-12 * np.max(np.abs(st["phi"]))
    assert np.max(np.abs(s["pi"] - st["pi"])) < 1e-12 * np.max(np.abs(st["pi"]))
    assert abs(s["a"] - st["a"]) == 0.0
    assert abs(s["b"] - st["b"]) < 1e-12 * st["b"]


@pytest.mark.parametrize("N", [32, 64, 96])
def test_two_field_initial_conditions_match_oracle_fp64(N):
    cfg = dict(synth.small(synth.config2(q=1000.0), N), precision="fp64")
    lat = _lattice(cfg)
    st = oracle.vacuum_ic(cfg)
    s = lat.get_state()
    for f in range(2):
        assert np.max(np.abs(s["phi"][f] - st["phi"][f])) < 1e-12 * np.max(np.abs(st["phi"][f]))
        assert np.max(np.abs(s["pi"][f] - st["pi"][f])) < 1e-12 * np.max(np.abs(st["pi"][f]))
    assert abs(s["b"] - st["b"]) < 1e-12 * st["b"]


# --------------------------------------------------------------------------
# configuration 2 physics: two fields, FP32 storage, VV2 and VV4
# --------------------------------------------------------------------------
@pytest.mark.parametrize("integ,q,nsteps", [("vv2", 100.0, 1000), ("vv4", 1000.0, 400), ("vv2", 1000.0, 1000),
                                             ("vv6", 100.0, 200), ("vv8", 100.0, 100), ("vv10", 1000.0, 40)])
def test_two_field_fp32_parity_64(integ, q, nsteps):
    cfg = synth.small(synth.config2(q=q, integrator=integ), 64)
    st = oracle.vacuum_ic(cfg)
    m = oracle.scalar_model(cfg)
    lat = _lattice(cfg)
    lat.set_state(st["phi"], st["pi"], st["a"], st["b"])
    phi, pi = st["phi"].copy(), st["pi"].copy()
    a, b = st["a"], st["b"]
    chunk = nsteps // 4
    worst = 0.0
    for k in range(4):
        lat.step(chunk)
        a, b = oracle.vv_steps(m, phi, pi, a, b, cfg["dt"], integ, chunk, omp=True)
        o = oracle.sync_observe(m, phi, pi, a, b)
        g = lat.energies()
        worst = max(worst, compare_obs(g, o, 2, 1e-5, f"{integ} step {chunk * (k + 1)}"))
    print(integ, q, "worst relative error", worst)


@pytest.mark.parametrize("alpha,integ", [(0.0, "vv2"), (0.5, "vv2"), (0.5, "vv4")])
def test_non_integer_alpha_fp64_parity(alpha, integ):
    # alpha-time other than conformal (Sec. 2.2, 4.1): the powers a^(k + m alpha)
    # of the drift, the kick and the expansion are then not all integers, and
    # the device forms the others with pow instead of by multiplication
    cfg = dict(synth.small(synth.config2(q=100.0, integrator=integ), 32), precision="fp64", alpha=alpha)
    st = oracle.vacuum_ic(cfg)
    m = oracle.scalar_model(cfg)
    lat = _lattice(cfg)
    lat.set_state(st["phi"], st["pi"], st["a"], st["b"])
    phi, pi = st["phi"].copy(), st["pi"].copy()
    lat.step(40)
    a, b = oracle.vv_steps(m, phi, pi, st["a"], st["b"], cfg["dt"], integ, 40)
    compare_obs(lat.energies(), oracle.sync_observe(m, phi, pi, a, b), 2, 1e-10, f"alpha {alpha} {integ}")
    s = lat.get_state()
    assert abs(s["a"] - a) < 1e-12 * a and a > st["a"]
    assert np.max(np.abs(s["phi"] - phi)) < 1e-10 * np.max(np.abs(phi))
    assert np.max(np.abs(s["pi"] - pi)) < 1e-10 * np.max(np.abs(pi))


@pytest.mark.parametrize("integ", ["vv6", "vv8", "vv10"])
def test_higher_order_yoshida_fp64_parity(integ):
    # VV6, VV8, VV10 (Sec. 3.4.1, 4.3.2): 7, 15, 31 fused passes per step
    cfg = dict(synth.small(synth.config2(q=100.0, integrator=integ), 32), precision="fp64")
    st = oracle.vacuum_ic(cfg)
    m = oracle.scalar_model(cfg)
    lat = _lattice(cfg)
    lat.set_state(st["phi"], st["pi"], st["a"], st["b"])
    phi, pi = st["phi"].copy(), st["pi"].copy()
    lat.step(24)
    a, b = oracle.vv_steps(m, phi, pi, st["a"], st["b"], cfg["dt"], integ, 24)
    compare_obs(lat.energies(), oracle.sync_observe(m, phi, pi, a, b), 2, 1e-10, integ)
    s = lat.get_state()
    assert np.max(np.abs(s["phi"] - phi)) < 1e-10 * np.max(np.abs(phi))
    assert np.max(np.abs(s["pi"] - pi)) < 1e-10 * np.max(np.abs(pi))


def test_ragged_size_96_fp32():
    cfg = synth.small(synth.config2(q=100.0), 96)
    st = oracle.vacuum_ic(cfg)
    m = oracle.scalar_model(cfg)
    lat = _lattice(cfg)
    lat.set_state(st["phi"], st["pi"], st["a"], st["b"])
    lat.step(60)
    phi, pi = st["phi"].copy(), st["pi"].copy()
    a, b = oracle.vv_steps(m, phi, pi, st["a"], st["b"], cfg["dt"], "vv2", 60, omp=True)
    compare_obs(lat.energies(), oracle.sync_observe(m, phi, pi, a, b), 2, 1e-5, "N=96")
    s = lat.get_state()
    assert np.max(np.abs(s["phi"] - phi)) < 2e-5 * np.max(np.abs(phi))


def _golden(case):
    import json
    import os

    path = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", f"full_size_{case}.json")
    with open(path) as f:
        return json.load(f)


def fp32_control(case):
    """Per-checkpoint errors of FP32 storage alone (FP64 oracle, state rounded
    to FP32 after every step) and of one FP32 rounding of the initial state,
    written by tests/golden/make_fp32_control.py; None where no control exists."""
    import json
    import os

    path = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", f"fp32_control_{case}.json")
    if not os.path.exists(path):
        return None
    with open(path) as f:
        return {cp["step"]: cp for cp in json.load(f)["checkpoints"]}


def window_end(ctl):
    """First checkpoint at which FP32 storage alone (the control) is 1e-6 or
    more away from the FP64 run on some observable.  Trajectory parity is gated
    at 1e-5 before it: a decade below the gate, since a kernel's FP32
    arithmetic adds rounding of the same order.  From there on the resonant
    growth of the fields amplifies any rounding a hundredfold per 100 steps or
    so, and no FP32 run can follow the FP64 one."""
    for step in sorted(ctl):
        if max(v for k, v in ctl[step]["storage"].items() if k != "gauss") >= 1e-6:
            return step
    return math.inf


@pytest.mark.parametrize("case", ["scalar2_256_vv2_q100", "scalar2_256_vv2_q1000", "scalar2_256_vv4_q1000"])
def test_full_size_256_window_against_stored_oracle_run(case):
    """Config 2 at 256^3 on the autotuned tile over 1000 steps (VV2, q = 100
    and 1000) and 300 steps (VV4), every 100 steps against the oracle's stored
    run (tests/golden/make_full_size.py), which is re-checked here against the
    live oracle at its initial state and at step 5.  Where an FP32 control
    exists (q = 100), the observables are gated at 1e-5 before its window end
    and the scale factor at every checkpoint; the other two runs stay inside
    the gate over their whole length."""
    gold = _golden(case)
    ctl = fp32_control(case)
    end = window_end(ctl) if ctl else math.inf
    cfg = dict(gold["config"])
    st = oracle.vacuum_ic(cfg)
    m = oracle.scalar_model(cfg)
    cps = {cp["step"]: cp["obs"] for cp in gold["checkpoints"]}
    o0 = oracle.sync_observe(m, st["phi"], st["pi"], st["a"], st["b"])
    for key in ("a", "b", "EK", "EG", "EV"):
        assert abs(o0[key] - cps[0][key]) <= 1e-13 * abs(cps[0][key]), key
    lat = _lattice(cfg)
    lat.set_state(st["phi"], st["pi"], st["a"], st["b"])
    phi, pi = st["phi"].copy(), st["pi"].copy()
    a, b = oracle.vv_steps(m, phi, pi, st["a"], st["b"], cfg["dt"], cfg["integrator"], 5, omp=True)
    o5 = oracle.sync_observe(m, phi, pi, a, b)
    del phi, pi
    for key in ("a", "b", "EK", "EG", "EV", "EK0", "EG1"):
        assert abs(o5[key] - cps[5][key]) <= 1e-12 * abs(cps[5][key]), key
    lat.step(5)
    compare_obs(lat.energies(), o5, 2, 1e-5, f"{case} step 5")
    done, worst, gated = 5, 0.0, 0
    for step in sorted(k for k in cps if k >= 100):
        lat.step(step - done)
        done = step
        g, o = lat.energies(), cps[step]
        if step < end:
            w = compare_obs(g, o, 2, 1e-5, f"{case} step {step}")
            worst = max(worst, w)
            gated += 1
            print(case, "step", step, "worst relative error %.2e" % w, flush=True)
        else:
            ea = abs(g["a"] - o["a"]) / o["a"]
            print(case, "step", step, "past the FP32 window: a %.1e" % ea, flush=True)
            assert ea < 1e-6, (step, ea)
    assert done == gold["nsteps"] and gated >= 3
    # pointwise values are not an observable of the method (late-time
    # fields are statistics, not gates): reported only
    s = lat.get_state()
    idx = tuple(np.array(i) for i in gold["sites"]["idx"])
    for key in ("phi", "pi"):
        ref = np.array(gold["sites"][key])
        d = np.max(np.abs(s[key][idx] - ref)) / np.max(np.abs(ref))
        print(case, key, "sampled sites, largest error relative to the largest value %.2e" % d, flush=True)
    print(case, "tile", lat.tiling(), "worst", worst)


def test_full_size_256_vv2_sampled_sites():
    cfg = synth.config2(q=100.0)
    st = oracle.vacuum_ic(cfg)
    m = oracle.scalar_model(cfg)
    lat = _lattice(cfg)
    lat.set_state(st["phi"], st["pi"], st["a"], st["b"])
    lat.step(5)
    phi, pi = st["phi"], st["pi"]
    a, b = oracle.vv_steps(m, phi, pi, st["a"], st["b"], cfg["dt"], "vv2", 5, omp=True)
    compare_obs(lat.energies(), oracle.sync_observe(m, phi, pi, a, b), 2, 1e-5, "256^3")
    s = lat.get_state()
    rng = np.random.default_rng(0)
    idx = (rng.integers(0, 2, size=4096),) + tuple(rng.integers(0, 256, size=(3, 4096)))
    for arr, ref in ((s["phi"], phi), (s["pi"], pi)):
        d = np.abs(arr[idx] - ref[idx])
        assert np.max(d) < 1e-5 * np.max(np.abs(ref[idx])), np.max(d)


def test_wide_tiles_256_against_oracle():
    """The z-wide tile shapes (128 and 256 threads along z) and the full-row
    tile over every x-chunk at 256^3, against the oracle after 5 steps."""
    cfg = synth.config2(q=100.0)
    st = oracle.vacuum_ic(cfg)
    m = oracle.scalar_model(cfg)
    phi, pi = st["phi"].copy(), st["pi"].copy()
    a, b = oracle.vv_steps(m, phi, pi, st["a"], st["b"], cfg["dt"], "vv2", 5, omp=True)
    o = oracle.sync_observe(m, phi, pi, a, b)
    lat = _lattice(cfg)
    rng = np.random.default_rng(2)
    idx = (rng.integers(0, 2, size=4096),) + tuple(rng.integers(0, 256, size=(3, 4096)))
    n = 0
    for (tz, by, ry) in ((128, 8, 2), (256, 4, 2), (128, 4, 2), (256, 8, 1)):
        for xc in (8, 16, 32, 64):
            lat.set_tiling(tz, by, ry, xc)
            lat.set_state(st["phi"], st["pi"], st["a"], st["b"])
            lat.step(5)
            compare_obs(lat.energies(), o, 2, 1e-5, f"tile {tz},{by},{ry},{xc}")
            s = lat.get_state()
            assert np.max(np.abs(s["phi"][idx] - phi[idx])) < 1e-5 * np.max(np.abs(phi[idx])), (tz, by, ry, xc)
            n += 1
    assert n == 16


def test_full_row_tiles_128_against_oracle():
    """The full-row tiles (a block holds whole z-rows, four sites per lane) at
    128^3 over every x-chunk down to 2 planes, against the oracle after 6 steps."""
    cfg = synth.small(synth.config2(q=100.0), 128)
    st = synth.random_state(cfg, seed=21, amp=0.3, mom=0.3)
    m = oracle.scalar_model(cfg)
    phi, pi = st["phi"].copy(), st["pi"].copy()
    a, b = oracle.vv_steps(m, phi, pi, 1.0, 0.5, cfg["dt"], "vv2", 6, omp=True)
    o = oracle.sync_observe(m, phi, pi, a, b)
    lat = _lattice(cfg)
    n = 0
    for (tz, by, ry) in ((128, 16, 1),):
        for xc in (2, 4, 8, 16, 32, 128):
            lat.set_tiling(tz, by, ry, xc)
            lat.set_state(st["phi"], st["pi"], 1.0, 0.5)
            lat.step(6)
            compare_obs(lat.energies(), o, 2, 1e-5, f"tile {tz},{by},{ry},{xc}")
            s = lat.get_state()
            assert np.max(np.abs(s["phi"] - phi)) < 1e-5 * np.max(np.abs(phi)), (tz, by, ry, xc)
            assert np.max(np.abs(s["pi"] - pi)) < 1e-5 * np.max(np.abs(pi)), (tz, by, ry, xc)
            n += 1
    assert n == 6


def test_full_row_tile_pass_is_bitwise_the_general_tiles():
    """One pass from the uploaded a and b (the leapfrog start-up kick): the
    full-row tiles do each site's arithmetic exactly as the general tile does,
    so the new fields and momenta agree bit for bit."""
    cfg = dict(synth.small(synth.config2(q=100.0), 256), integrator="lf2")
    st = synth.random_state(cfg, seed=22, amp=0.3, mom=0.3)
    lat = _lattice(cfg)
    out = []
    for t in ((128, 8, 2, 32), (256, 8, 1, 16), (256, 8, 1, 32), (256, 8, 1, 64)):
        lat.set_tiling(*t)
        lat.set_state(st["phi"], st["pi"], 1.0, 0.5)
        lat.step(0)
        out.append(lat.get_state())
    for k, s in enumerate(out[1:]):
        assert np.array_equal(s["phi"], out[0]["phi"]), k
        assert np.array_equal(s["pi"], out[0]["pi"]), k


def test_full_row_tiles_fp64_against_oracle():
    """FP64 storage (two sites per lane) on the full-row tiles: 128^3 over
    several x-chunks and 256^3 on the 256 x 4 tile, against the oracle at the
    FP64 tolerance."""
    for N, shape, xcs, nsteps in ((128, (128, 8, 1), (2, 8, 32, 128), 6), (256, (256, 4, 1), (32,), 3)):
        cfg = dict(synth.small(synth.config2(q=100.0), N), precision="fp64")
        st = synth.random_state(cfg, seed=23, amp=0.3, mom=0.3)
        m = oracle.scalar_model(cfg)
        phi, pi = st["phi"].copy(), st["pi"].copy()
        a, b = oracle.vv_steps(m, phi, pi, 1.0, 0.5, cfg["dt"], "vv2", nsteps, omp=True)
        o = oracle.sync_observe(m, phi, pi, a, b)
        lat = _lattice(cfg)
        for xc in xcs:
            lat.set_tiling(*shape, xc)
            lat.set_state(st["phi"], st["pi"], 1.0, 0.5)
            lat.step(nsteps)
            compare_obs(lat.energies(), o, 2, 1e-10, f"fp64 tile {shape},{xc}")
            s = lat.get_state()
            assert np.max(np.abs(s["phi"] - phi)) < 1e-10 * np.max(np.abs(phi)), (N, xc)
            assert np.max(np.abs(s["pi"] - pi)) < 1e-10 * np.max(np.abs(pi)), (N, xc)
        lat.close()


@pytest.mark.parametrize("precision, shape, tol", [("fp32", (128, 16, 1), 1e-5), ("fp64", (128, 8, 1), 1e-10)])
def test_full_row_tiles_lf2_against_oracle(precision, shape, tol):
    """Staggered leapfrog on the full-row tiles (the start-up kick, then
    drift + kick passes with the kinetic term of the half-step momenta) at
    128^3, against the oracle's scheme III at two checkpoints."""
    cfg = dict(synth.small(synth.config2(q=100.0, integrator="lf2"), 128), precision=precision)
    st = synth.random_state(cfg, seed=25, amp=0.3, mom=0.3)
    m = oracle.scalar_model(cfg)
    lat = _lattice(cfg)
    lat.set_tiling(*shape, 16)
    lat.set_state(st["phi"], st["pi"], 1.0, 0.5)
    phi, pi = st["phi"].copy(), st["pi"].copy()
    h = cfg["dt"]
    a, b = oracle.lf_startup(m, phi, pi, 1.0, 0.5, h)
    for k in range(2):
        lat.step(4)
        a, b = oracle.lf_steps(m, phi, pi, a, b, h, 4, omp=True)
        compare_obs(lat.energies(), oracle.lf_observe(m, phi, pi, a, b, h), 2, tol, f"{precision} lf2 {4 * (k + 1)}")
    s = lat.get_state()
    assert s["staggered"]
    assert np.max(np.abs(s["phi"] - phi)) < tol * np.max(np.abs(phi))
    assert np.max(np.abs(s["pi"] - pi)) < tol * np.max(np.abs(pi))


def test_full_row_tile_fp64_512_sampled_sites():
    # the 512 x 2 full-row tile (two rows per block, two sites per lane)
    cfg = dict(synth.config2(q=100.0, N=512), precision="fp64")
    st = oracle.vacuum_ic(cfg)
    m = oracle.scalar_model(cfg)
    lat = _lattice(cfg)
    lat.set_tiling(512, 2, 1, 32)
    lat.set_state(st["phi"], st["pi"], st["a"], st["b"])
    lat.step(2)
    phi, pi = st["phi"], st["pi"]
    a, b = oracle.vv_steps(m, phi, pi, st["a"], st["b"], cfg["dt"], "vv2", 2, omp=True)
    compare_obs(lat.energies(), oracle.sync_observe(m, phi, pi, a, b), 2, 1e-10, "512^3 fp64 rows")
    s = lat.get_state()
    rng = np.random.default_rng(3)
    idx = (rng.integers(0, 2, size=4096),) + tuple(rng.integers(0, 512, size=(3, 4096)))
    for arr, ref in ((s["phi"], phi), (s["pi"], pi)):
        assert np.max(np.abs(arr[idx] - ref[idx])) < 1e-10 * np.max(np.abs(ref[idx]))
    lat.close()


def test_full_row_tile_fp64_pass_is_bitwise_the_general_tiles():
    cfg = dict(synth.small(synth.config2(q=100.0), 256), integrator="lf2", precision="fp64")
    st = synth.random_state(cfg, seed=24, amp=0.3, mom=0.3)
    lat = _lattice(cfg)
    out = []
    for t in ((32, 8, 2, 32), (256, 4, 1, 16), (256, 4, 1, 64)):
        lat.set_tiling(*t)
        lat.set_state(st["phi"], st["pi"], 1.0, 0.5)
        lat.step(0)
        out.append(lat.get_state())
    for k, s in enumerate(out[1:]):
        assert np.array_equal(s["phi"], out[0]["phi"]), k
        assert np.array_equal(s["pi"], out[0]["pi"]), k


def test_large_512_vv2_sampled_sites():
    cfg = synth.config2(q=100.0, N=512)
    st = oracle.vacuum_ic(cfg)
    m = oracle.scalar_model(cfg)
    lat = _lattice(cfg)
    lat.set_state(st["phi"], st["pi"], st["a"], st["b"])
    lat.step(2)
    phi, pi = st["phi"], st["pi"]
    a, b = oracle.vv_steps(m, phi, pi, st["a"], st["b"], cfg["dt"], "vv2", 2, omp=True)
    compare_obs(lat.energies(), oracle.sync_observe(m, phi, pi, a, b), 2, 1e-5, "512^3")
    s = lat.get_state()
    rng = np.random.default_rng(1)
    idx = (rng.integers(0, 2, size=4096),) + tuple(rng.integers(0, 512, size=(3, 4096)))
    for arr, ref in ((s["phi"], phi), (s["pi"], pi)):
        d = np.abs(arr[idx] - ref[idx])
        assert np.max(d) < 1e-5 * np.max(np.abs(ref[idx])), np.max(d)


def test_max_size_1024_device_state_steps():
    # The largest supported lattice, from device initial conditions.  With the
    # literal vacuum amplitude the fluctuation energy dominates at 1024^3 and
    # the expansion is fast (a grows several-fold in a few steps), so the
    # Hubble-constraint residual is not small; it must still fall at least as
    # dt^2 at fixed eta (VV2), which checks the coupled field/scale-factor
    # update at this size.
    import torch
    hc = []
    # the vacuum energy makes H ~ 10^2 here: steps small enough that dt H << 1
    for dt, n in ((0.001, 20), (0.0005, 40)):
        cfg = dict(synth.config2(q=100.0, N=1024), dt=dt)
        lat = _lattice(cfg)
        a0 = lat.energies()["a"]
        lat.step(n)
        e = lat.energies()
        assert all(math.isfinite(e[k]) for k in ("a", "b", "EK", "EG", "EV", "hc"))
        assert e["a"] > a0 and e["step"] == n and abs(e["eta"] - 0.02) < 1e-12
        hc.append(e["hc"])
        lat.close()
        del lat
        torch.cuda.empty_cache()
    # at least second order (the paper's statement for VV2); over this short
    # interval the measured ratio is 8, the third-order local error of the
    # first steps still dominating
    assert 3.0 < hc[0] / hc[1] < 9.0, hc


def test_every_tiling_agrees():
    cfg = synth.small(synth.config2(q=300.0), 64)
    st = synth.random_state(cfg, seed=7, amp=0.3, mom=0.3)
    m = oracle.scalar_model(cfg)
    phi, pi = st["phi"].copy(), st["pi"].copy()
    a, b = oracle.vv_steps(m, phi, pi, 1.0, 0.5, cfg["dt"], "vv2", 8, omp=True)
    o = oracle.sync_observe(m, phi, pi, a, b)
    lat = _lattice(cfg)
    shapes = [(64, 4, 2), (64, 8, 2), (32, 8, 2)]
    n = 0
    for (tz, by, ry) in shapes:
        for xc in (4, 8, 16, 32):
            try:
                lat.set_tiling(tz, by, ry, xc)
            except Exception:
                continue
            lat.set_state(st["phi"], st["pi"], 1.0, 0.5)
            lat.step(8)
            compare_obs(lat.energies(), o, 2, 1e-5, f"tile {tz},{by},{ry},{xc}")
            s = lat.get_state()
            assert np.max(np.abs(s["phi"] - phi)) < 1e-5 * np.max(np.abs(phi)), (tz, by, ry, xc)
            n += 1
    assert n == 12


@pytest.mark.parametrize("precision,nf,N,shapes", [
    ("fp32", 2, 32, ((8, 4), (16, 2), (8, 32))), ("fp32", 2, 96, ((8, 3), (16, 1), (16, 96))),
    ("fp32", 2, 160, ((16, 5),)), ("fp32", 1, 96, ((8, 2), (16, 48))), ("fp64", 2, 32, ((4, 8), (8, 4))),
    ("fp64", 2, 96, ((4, 3), (8, 96))), ("fp64", 2, 160, ((8, 8),)), ("fp64", 1, 64, ((2, 8), (8, 2)))])
def test_full_row_tiles_of_any_length_against_oracle(precision, nf, N, shapes):
    """Full-row tiles where a row is no power of two, a block is one wave or
    twelve, holds the whole plane or marches the whole lattice; one leapfrog
    start-up kick is bit for bit the general tile's, five steps agree with the
    oracle."""
    base = synth.config2(q=100.0) if nf == 2 else dict(synth.config2(q=100.0), nf=1, q=0.0)
    cfg = dict(synth.small(base, N), precision=precision)
    st = synth.random_state(cfg, seed=31, amp=0.3, mom=0.3)
    m = oracle.scalar_model(cfg)
    phi, pi = st["phi"].copy(), st["pi"].copy()
    a, b = oracle.vv_steps(m, phi, pi, 1.0, 0.5, cfg["dt"], "vv2", 5, omp=True)
    tol = 1e-5 if precision == "fp32" else 1e-10
    lat, kick = _lattice(cfg), _lattice(dict(cfg, integrator="lf2"))
    ref = None
    for t in [(32, 8, 2, 8)] + [(N, by, 1, xc) for by, xc in shapes]:
        kick.set_tiling(*t)
        kick.set_state(st["phi"], st["pi"], 1.0, 0.5)
        kick.step(0)
        s = kick.get_state()
        ref = ref or s
        assert np.array_equal(s["phi"], ref["phi"]) and np.array_equal(s["pi"], ref["pi"]), t
        lat.set_tiling(*t)
        lat.set_state(st["phi"], st["pi"], 1.0, 0.5)
        lat.step(5)
        compare_obs(lat.energies(), oracle.sync_observe(m, phi, pi, a, b), nf, tol, f"{t}")
        s = lat.get_state()
        assert np.max(np.abs(s["phi"] - phi)) < tol * np.max(np.abs(phi)), t
        assert np.max(np.abs(s["pi"] - pi)) < tol * np.max(np.abs(pi)), t


@pytest.mark.parametrize("integ", ["lf2", "vv2"])
@pytest.mark.parametrize("nf,N,by,xc", [(2, 64, 4, 4), (2, 96, 8, 8), (2, 160, 8, 16), (1, 64, 16, 8), (1, 96, 8, 4),
                                        (1, 32, 8, 4)])
def test_full_row_sums_carry_the_bits_of_the_general_tile(nf, N, by, xc, integ):
    """A full-row tile adds each FP32 site's terms to the FP64 sums one by one,
    as the general tile does: a and b agree to the order of the FP64 additions.
    The four sites of a lane hold different values, the same in every lane, so
    that terms added in FP32 first (rounded by up to 6e-8) would not average
    out.  The potential is a mass term, whose rounding is the same in both
    tiles.  64^3 to 160^3 additions of equal sign in another order differ by at
    most 1e-11 of b's change (1e-13 in practice); each a and b carries 1e-16 of
    itself."""
    cfg = dict(synth.small(synth.config2(q=0.0), N), nf=nf, integrator=integ, m2=(0.5, 0.0), lam=0.0, alpha=0.0,
               fstar_over_mp=1.0)
    rng = np.random.default_rng(100 * N + by)
    four = rng.uniform(0.3, 1.0, (2, nf, 4)).astype(np.float32).astype(np.float64)
    phi, pi = np.broadcast_to(np.tile(four, N // 4)[:, :, None, None, :], (2, nf, N, N, N)).copy()
    lat = _lattice(cfg)
    out = []
    for t in ((32, 8, 2, 8), (N, by, 1, xc)):
        lat.set_tiling(*t)
        lat.set_state(phi, pi, 1.0, 0.5)
        lat.step(2)
        out.append(lat.get_state())
    g, r = out
    for k, start in (("a", 1.0), ("b", 0.5)):
        assert abs(r[k] - g[k]) < 1e-11 * abs(g[k] - start) + 1e-15 * abs(g[k]), (k, (r[k] - g[k]) / (g[k] - start))
    lat.close()


def full_row_planes(N, width, by, xc):
    """Planes of each block along x that a full-row pass marches: the fewest
    blocks of at most xc planes, or more, of eight planes or one per CU, where
    the GPU then ends sooner (twelve waves share a CU)."""
    slots = 256 * max(1, 12 // (N // width * by // 64))
    tiles, n, best, cost = N // by, N // xc, 0, math.inf
    n0 = n
    while n == n0 or 8 * n <= N or (n <= N and tiles * n <= 256):
        c = -(-tiles * n // slots) * (-(-N // n) + 2.0)
        if c < 0.98 * cost:
            cost, best = c, n
        n += 1
    return sorted({(k + 1) * N // best - k * N // best for k in range(best)})


@pytest.mark.parametrize("precision,N,by,xc,lanes,lds,planes", [
    ("fp32", 192, 16, 192, 768, 55296, [9, 10]), ("fp64", 192, 8, 64, 768, 61440, [19, 20]),
    ("fp32", 384, 8, 32, 768, 61440, [24]), ("fp64", 384, 4, 48, 768, 73728, [48]),
    ("fp32", 768, 4, 96, 768, 73728, [96]), ("fp64", 32, 4, 32, 64, 6144, [1])])
def test_full_row_blocks_at_their_bounds(precision, N, by, xc, lanes, lds, planes):
    """The largest full-row blocks, 768 lanes and up to 72 KB of LDS, and one
    wave: a start-up kick is bit for bit the general tile's at every site, two
    leapfrog steps agree to a few roundings of the state (a and b differ by the
    order of FP64 additions), and the observation's kinetic sum and means are
    the device's own in FP64."""
    import torch
    from test_gpu_u1 import component

    width = 4 if precision == "fp32" else 2
    assert lanes == N // width * by and lds == 2 * 2 * (by + 2) * N * 16 // width
    assert full_row_planes(N, width, by, xc) == planes
    cfg = dict(synth.config2(q=100.0, N=N), precision=precision, integrator="lf2", ic="homogeneous")
    out = []
    for t in ((32, 8, 2, 8), (N, by, 1, xc)):
        lat = _lattice(cfg)
        lat.set_tiling(*t)
        g = torch.Generator(device="cuda:0").manual_seed(N)
        for c in range(4):
            d = component(lat, c)
            d.copy_(0.3 * torch.rand(d.shape, generator=g, device=d.device, dtype=d.dtype))
        torch.cuda.synchronize()
        e = lat.energies()
        for f in range(2):
            p = component(lat, 2 + f)
            ek = float((p * p).double().mean()) / 2.0 / e["a"] ** 6
            assert abs(e[f"EK{f}"] - ek) < 1e-11 * ek and abs(
                e[f"mean{f}"] - float(component(lat, f).double().mean())) < 1e-11, (t, f)
        lat.step(0)
        torch.cuda.synchronize()
        kick = [component(lat, c).clone() for c in range(4)]
        lat.step(2)
        torch.cuda.synchronize()
        out.append((kick, [component(lat, c).clone() for c in range(4)]))
        lat.close()
        del lat, d, p
        torch.cuda.empty_cache()
    eps = 1.2e-7 if precision == "fp32" else 2.3e-16
    for c in range(4):
        assert torch.equal(out[0][0][c], out[1][0][c]), c
        a, b = out[0][1][c], out[1][1][c]
        assert float((a - b).abs().max()) <= 8 * eps * float(a.abs().max()), c


@pytest.mark.parametrize("N", [32, 96, 160])
def test_spectrum_of_single_modes_on_the_half_volume(N):
    """The transform keeps half the modes along z and counts the others through
    their conjugates: single plane waves on its seams (n3 = 0 and N/2, which
    share storage, n1 or n2 = 0 and N/2, self-conjugate corners) each put their
    whole power, N^6/2 for a cosine and N^6 for a self-conjugate mode, into
    their own shell."""
    cfg = dict(synth.small(synth.config2(q=100.0), N), precision="fp64")
    lat = _lattice(cfg)
    h = N // 2
    n = np.arange(N)
    zero = np.zeros((2, N, N, N))
    for m in ((0, 0, 0), (3, 5, 0), (0, 0, 4), (h, 0, 0), (0, h, 0), (0, 0, h), (h, h, h), (h, 0, 7), (2, h, h),
              (-2, 4, h - 1), (5, -3, h), (1, 0, h), (0, 2, 0), (-7, h, 0)):
        ph = 2.0 * np.pi * ((m[0] * n[:, None, None] + m[1] * n[:, None] + m[2] * n) % N) / N
        phi = zero.copy()
        phi[1] = np.cos(ph)
        lat.set_state(phi, zero, 1.0, 0.5)
        s = lat.spectrum(1)["S"]
        sh = int(math.isqrt(sum(k * k for k in m)))
        selfconj = all(k % h == 0 for k in m)
        assert abs(s[sh] / (N ** 6 * (1.0 if selfconj else 0.5)) - 1.0) < 1e-12, (m, s[sh] / N ** 6)
        assert np.sum(np.delete(s, sh)) < 1e-24 * N ** 6, m
    lat.close()


def test_bitwise_determinism():
    cfg = synth.small(synth.config2(q=100.0), 64)
    st = synth.random_state(cfg, seed=3)
    out = []
    for _ in range(2):
        lat = _lattice(cfg)
        lat.set_state(st["phi"], st["pi"], 1.0, 0.4)
        lat.step(20)
        out.append((lat.get_state(), lat.energies()))
        lat.close()
    assert np.array_equal(out[0][0]["phi"], out[1][0]["phi"])
    assert np.array_equal(out[0][0]["pi"], out[1][0]["pi"])
    assert out[0][1]["EK"] == out[1][1]["EK"] and out[0][0]["b"] == out[1][0]["b"]


def test_lf_resume_and_checkpoint():
    cfg = synth.config1()
    st = oracle.vacuum_ic(cfg)
    lat = _lattice(cfg)
    lat.set_state(st["phi"], st["pi"], st["a"], st["b"])
    lat.step(7)
    ref = lat.get_state()
    lat2 = _lattice(cfg)
    lat2.set_state(st["phi"], st["pi"], st["a"], st["b"])
    lat2.step(3)
    ck = lat2.get_state()
    lat3 = _lattice(cfg)
    lat3.set_state(ck["phi"], ck["pi"], ck["a"], ck["b"], eta=ck["eta"], step=ck["step"],
                   staggered=ck["staggered"])
    lat3.step(4)
    s = lat3.get_state()
    assert s["step"] == 7
    assert np.max(np.abs(s["phi"] - ref["phi"])) < 1e-13
    assert abs(s["a"] - ref["a"]) < 1e-14


def test_zero_steps_and_energies_idempotent():
    cfg = synth.small(synth.config2(), 32)
    lat = _lattice(cfg)
    s0 = lat.get_state()
    lat.step(0)
    e1, e2 = lat.energies(), lat.energies()
    s1 = lat.get_state()
    assert set(e1) == set(e2)
    for k in e1:
        assert e1[k] == e2[k] or (isinstance(e1[k], float) and math.isnan(e1[k]) and math.isnan(e2[k])), k
    assert np.array_equal(s0["phi"], s1["phi"])


def test_flat_space_free_mode_dispersion_on_gpu():
    # the exact lattice dispersion of a free massive mode, through the HIP path
    N, m2, h, nsteps = 32, 0.37, 0.05, 40
    cfg = dict(model="scalar", nf=1, N=N, kIR=0.7, dt=h, alpha=1.0, fstar_over_mp=1.0, m2=(m2, 0.0),
               lam=0.0, q=0.0, expansion=False, integrator="vv2", precision="fp64", ic="homogeneous",
               phi0=(0.0, 0.0))
    dx = 2 * math.pi / (0.7 * N)
    nvec = (3, 5, 7)
    w2 = m2 + sum((2.0 / dx * math.sin(math.pi * n / N)) ** 2 for n in nvec)
    x = np.arange(N)
    X, Y, Z = np.meshgrid(x, x, x, indexing="ij")
    mode = np.cos(2 * math.pi * (nvec[0] * X + nvec[1] * Y + nvec[2] * Z) / N + 0.2)
    lat = _lattice(cfg)
    lat.set_state((0.8 * mode)[None], (-0.3 * mode)[None], 1.0, 0.0)
    lat.step(nsteps)
    M = np.array([[1 - h * h * w2 / 2, h], [-h * w2 * (1 - h * h * w2 / 4), 1 - h * h * w2 / 2]])
    A, B = np.linalg.matrix_power(M, nsteps) @ np.array([0.8, -0.3])
    s = lat.get_state()
    assert np.max(np.abs(s["phi"][0] - A * mode)) < 1e-12
    assert np.max(np.abs(s["pi"][0] - B * mode)) < 1e-11


@pytest.mark.parametrize("precision,N", [("fp64", 32), ("fp64", 64), ("fp32", 96), ("fp32", 128), ("fp32", 160),
                                         ("fp32", 224), ("fp32", 256), ("fp32", 384)])
def test_spectrum_matches_oracle(precision, N):
    # 96, 160 and 224 take the radix-3, radix-5 and generic (radix-7) FFT
    # stages; the binning pass factors 128, 256 and 384 as 8 8 2, 8 8 4 and
    # 8 8 2 3 (the other passes in radices 4 and 2); 256 is the benchmarked
    # size; above 256 the binning pass keeps four times the shell histograms
    # (one field there: the oracle's transform of 384^3 takes seconds)
    cfg = dict(synth.small(synth.config2(q=100.0), N), precision=precision)
    lat = _lattice(cfg)
    s = lat.get_state()
    tol = 1e-10 if precision == "fp64" else 1e-5
    cases = ((0, s["phi"][0]), (1, s["phi"][1]), (17, s["pi"][1]))
    for which, arr in cases[:1] if N > 256 else cases:
        g = lat.spectrum(which)
        o = oracle.spectrum(arr, cfg["kIR"])
        assert np.array_equal(g["count"], o["count"])
        # mean |k| of a shell: the oracle sums its n modes' |k| one after
        # another in FP64 (relative error up to (n - 1) eps; n reaches 1e6
        # at 384^3), the device in per-block partial sums (smaller)
        kt = 2.0 * np.finfo(np.float64).eps * np.maximum(o["count"], 1) * np.abs(o["k"])
        assert np.all(np.abs(g["k"] - o["k"]) <= kt), np.max(np.abs(g["k"] - o["k"]) / np.maximum(kt, 1e-300))
        check_shells(g, o, tol, f"{precision} N={N} which={which}")


def test_nonfinite_state_rejected():
    from paper_2006_15122_amd.lattice import LatticeError

    cfg = synth.small(synth.config2(), 32)
    lat = _lattice(cfg)
    st = synth.random_state(cfg, seed=1)
    st["phi"][0, 1, 2, 3] = np.nan
    with pytest.raises(LatticeError) as e:
        lat.set_state(st["phi"], st["pi"], 1.0, 0.1)
    assert "LAT_ENONFINITE" in str(e.value)


def test_hubble_constraint_ladder_of_the_verlet_family():
    """The paper's integrator comparison (Sec. 8.2.1): the Hubble-constraint
    violation falls by orders of magnitude from VV2 up to VV10, until round-off
    stops it, and the staggered leapfrog is no worse than VV2.  Two fields,
    q = 100, 64^3, FP64 storage, eta = 20."""
    from paper_2006_15122_amd.lattice import Lattice

    dt, eta = 0.005, 20.0
    n = int(round(eta / dt))
    hc = {}
    for integ in ("lf2", "vv2", "vv4", "vv6", "vv8", "vv10"):
        cfg = dict(synth.small(synth.config2(q=100.0, integrator=integ), 64), precision="fp64", dt=dt)
        lat = Lattice(cfg, device="cuda:0")
        lat.step(n)
        hc[integ] = lat.energies()["hc"]
        lat.close()
        print(integ, "hubble-constraint violation %.3e" % hc[integ], flush=True)
    assert hc["lf2"] <= hc["vv2"]
    order = ("vv2", "vv4", "vv6", "vv8", "vv10")
    floor = 1e-13
    for lo, hi in zip(order, order[1:]):
        # each order at least tenfold below the previous one, unless the
        # previous one has already reached the round-off floor
        assert hc[hi] <= max(hc[lo] / 10.0, 10 * floor), (lo, hi, hc[lo], hc[hi])
    assert hc["vv2"] / max(hc["vv10"], floor) > 1e6


def test_integrator_orders_from_the_hubble_constraint():
    """Each integrator's order (Sec. 3.4, 4.2, 4.3), read off the
    Hubble-constraint violation at eta = 20: halving the step from 0.01 to
    0.005 divides it by 2^p within a factor 1.5 (p = 2 for the staggered
    leapfrog and VV2, 4 and 6 for VV4 and VV6); VV8 and VV10 are at the
    round-off floor by then.  Two fields, q = 100, 32^3, FP64 storage."""
    from paper_2006_15122_amd.lattice import Lattice

    eta = 20.0
    hc = {}
    for dt in (0.01, 0.005):
        for integ in ("lf2", "vv2", "vv4", "vv6", "vv8", "vv10"):
            cfg = dict(synth.small(synth.config2(q=100.0, integrator=integ), 32), precision="fp64", dt=dt)
            lat = Lattice(cfg, device="cuda:0")
            lat.step(int(round(eta / dt)))
            hc[dt, integ] = lat.energies()["hc"]
            lat.close()
            print(f"dt {dt} {integ}: hubble-constraint violation {hc[dt, integ]:.3e}", flush=True)
    for integ, p in (("lf2", 2), ("vv2", 2), ("vv4", 4), ("vv6", 6)):
        r = hc[0.01, integ] / hc[0.005, integ]
        assert 2.0 ** p / 1.5 < r < 2.0 ** p * 1.5, (integ, p, r)
    assert hc[0.005, "vv8"] < 1e-13 and hc[0.005, "vv10"] < 1e-13


def test_two_full_size_inits_are_bitwise_equal():
    # the tuner's pick is kept per configuration, so a second 256^3 lattice of the
    # same workload takes the same tile and reproduces the first bit for bit
    cfg = synth.config2(q=100.0)
    out = []
    for _ in range(2):
        lat = _lattice(cfg)
        lat.step(20)
        out.append((lat.tiling(), lat.energies(), lat.get_state()))
        lat.close()
    assert out[0][0] == out[1][0]
    for k in ("a", "b", "EK", "EG", "EV"):
        assert out[0][1][k] == out[1][1][k], k
    assert np.array_equal(out[0][2]["phi"], out[1][2]["phi"])
    assert np.array_equal(out[0][2]["pi"], out[1][2]["pi"])
