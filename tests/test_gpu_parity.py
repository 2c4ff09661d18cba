"""GPU parity tests: every kernel of the path, called through the C ABI,
against the CPU oracle on the same seeded inputs.

Tolerances: positions within 1e-10 au after a year of integration; the
light-time direction from a given state within 1e-12 rad; pair sets
identical except pairs whose oracle edge distance is below 1 mas."""
import dataclasses
import math
import sys

import numpy as np
import pytest

from paper_2509_04666_amd import synth

pytestmark = pytest.mark.gpu

MAS = math.radians(1.0 / 3.6e6)


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2509_04666_amd import api
    return torch, api


def _say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def _dev_x(torch, x):
    return torch.as_tensor(np.ascontiguousarray(x), dtype=torch.float64).cuda()


# ---------------------------------------------------------------- ephemeris
def test_ephem_eval_matches_oracle(torch_cuda, orc):
    torch, api = torch_cuda
    case = synth.survey_case(n_obj=1, n_frames=0)
    e = case.ephem
    rng = np.random.default_rng(11)
    joints = e.t_start + e.seg_days * np.arange(1, e.n_seg)
    t = np.concatenate([rng.uniform(e.t_start, e.t_end, 300), joints, [e.t_start, e.t_end]])
    out = api.ephem_eval(api.DeviceEphemeris.from_synth(e), t).cpu().numpy()
    err_p = err_v = 0.0
    for q, tq in enumerate(t):
        for b in range(e.n_body):
            st, p, v = orc.cheb(e, b, tq)
            assert st == 0
            err_p = max(err_p, np.max(np.abs(out[q, b, :3] - p)))
            err_v = max(err_v, np.max(np.abs(out[q, b, 3:] - v)))
    _say(f"ephem max |dp| {err_p:.3e} au, |dv| {err_v:.3e} au/d")
    assert err_p < 1e-13 and err_v < 1e-14


# ---------------------------------------------------------------- light time
def test_lighttime_matches_oracle(torch_cuda, orc):
    torch, api = torch_cuda
    case = synth.survey_case(n_obj=300, n_frames=0, neo_frac=0.2)
    rng = np.random.default_rng(12)
    t_ref = 40.0
    xs, st, _ = orc.propagate(case.ephem, case.x0, 0.0, [t_ref])
    states = xs[0]
    t_obs = t_ref + rng.uniform(-1.6, 1.6, 12)
    obs = synth.circular_observer(case.model, t_obs)
    eph = api.DeviceEphemeris.from_synth(case.ephem)
    d, tau = api.lighttime_directions(eph, _dev_x(torch, states), t_ref, _dev_x(torch, t_obs), _dev_x(torch, obs))
    d = d.cpu().numpy(); tau = tau.cpu().numpy()
    worst_ang = worst_tau = 0.0
    for q in range(t_obs.size):
        dref, tref = orc.directions(case.ephem, states, t_ref, t_obs[q], obs[q])
        cosang = np.sum(d[q] * dref, 1) / np.linalg.norm(d[q], axis=1) / np.linalg.norm(dref, axis=1)
        ang = np.arccos(np.clip(cosang, -1, 1))
        cr = np.linalg.norm(np.cross(d[q], dref), axis=1) / np.linalg.norm(d[q], axis=1) / np.linalg.norm(dref, axis=1)
        worst_ang = max(worst_ang, np.max(np.minimum(ang, cr)))
        worst_tau = max(worst_tau, np.max(np.abs(tau[q] - tref)))
        np.testing.assert_allclose(d[q], dref, rtol=0, atol=1e-13)
    _say(f"light-time max angle {worst_ang:.3e} rad, max |dtau| {worst_tau:.3e} d")
    assert worst_ang < 1e-12 and worst_tau < 1e-15


def test_lighttime_extreme_geometries(torch_cuda, orc):
    """Bodies far and near, slow and fast, and hops of up to 8 days: distant
    (40 au) and very distant (400 au) bodies, bodies 0.002 au from the
    observer, a Sun-grazer near perihelion and fast hyperbolic bodies.  The
    light time reaches 2.3 days for the farthest; the directions must match
    the oracle's plain iteration to the same bar as the survey bodies."""
    torch, api = torch_cuda
    case = synth.survey_case(n_obj=1, n_frames=0)
    rng = np.random.default_rng(13)
    t_ref = 40.0
    gm = synth.GM_SUN
    sun = case.model.sun(np.array([t_ref]))[0]
    rows = []
    def add(r, v):
        rows.append(np.concatenate([np.asarray(r, float) + sun[:3], np.asarray(v, float) + sun[3:]]))
    for dist in (40.0, 400.0):
        for _ in range(8):
            u = rng.normal(size=3); u /= np.linalg.norm(u)
            w = np.cross(u, rng.normal(size=3)); w /= np.linalg.norm(w)
            add(dist * u, math.sqrt(gm / dist) * w * rng.uniform(0.5, 1.3))
    for _ in range(8):                                   # fast hyperbolic bodies at 1-3 au
        u = rng.normal(size=3); u /= np.linalg.norm(u)
        w = rng.normal(size=3); w /= np.linalg.norm(w)
        add(rng.uniform(1.0, 3.0) * u, rng.uniform(0.03, 0.08) * w)
    for _ in range(4):                                   # Sun-grazers near perihelion
        u = rng.normal(size=3); u /= np.linalg.norm(u)
        w = np.cross(u, rng.normal(size=3)); w /= np.linalg.norm(w)
        q = rng.uniform(0.02, 0.1)
        add(q * u, math.sqrt(1.9 * gm / q) * w)
    t_obs = t_ref + np.concatenate([rng.uniform(-8.0, 8.0, 6), [0.0, 1e-9]])
    obs = synth.circular_observer(case.model, t_obs)
    o_ref = synth.circular_observer(case.model, np.array([t_ref]))[0]
    for _ in range(6):                                   # bodies 0.002 au from the observer at t_ref
        u = rng.normal(size=3); u /= np.linalg.norm(u)
        w = rng.normal(size=3); w /= np.linalg.norm(w)
        rows.append(np.concatenate([o_ref + 0.002 * u, sun[3:] + 0.02 * w]))
    states = np.array(rows)
    eph = api.DeviceEphemeris.from_synth(case.ephem)
    d, tau = api.lighttime_directions(eph, _dev_x(torch, states), t_ref, _dev_x(torch, t_obs), _dev_x(torch, obs))
    d = d.cpu().numpy(); tau = tau.cpu().numpy()
    worst_ang = worst_tau = 0.0
    for q in range(t_obs.size):
        dref, tref = orc.directions(case.ephem, states, t_ref, t_obs[q], obs[q])
        assert np.all(np.isfinite(dref)) and np.all(np.isfinite(d[q]))
        n1, n2 = np.linalg.norm(d[q], axis=1), np.linalg.norm(dref, axis=1)
        cr = np.linalg.norm(np.cross(d[q], dref), axis=1) / n1 / n2
        worst_ang = max(worst_ang, float(np.max(cr)))
        worst_tau = max(worst_tau, float(np.max(np.abs(tau[q] - tref))))
        np.testing.assert_allclose(d[q], dref, rtol=1e-14, atol=1e-13)
    _say(f"light-time (extreme geometries) max angle {worst_ang:.3e} rad, max |dtau| {worst_tau:.3e} d, "
         f"max tau {tau.max():.3f} d")
    assert worst_ang < 1e-12 and worst_tau < 3e-15


# ---------------------------------------------------------------- propagation
def _propagate_both(torch, api, orc, ephem, x0, t0, t_out, **opts):
    eph = api.DeviceEphemeris.from_synth(ephem)
    o = api.default_opts(**opts)
    xg, sg = api.propagate(eph, _dev_x(torch, x0), t0, t_out, o)
    xo, so, _ = orc.propagate(ephem, x0, t0, t_out)
    return xg.cpu().numpy(), sg.cpu().numpy(), xo, so


def test_propagate_sun_only_one_year(torch_cuda, orc):
    torch, api = torch_cuda
    rng = np.random.default_rng(13)
    el = np.concatenate([synth.main_belt_elements(rng, 200), synth.neo_elements(rng, 56)])
    x0 = synth.elements_to_state(*[el[:, k] for k in range(6)], synth.GM_SUN)
    eph = synth.sun_only_ephemeris(-8.0, 60)
    t_out = np.arange(30.0, 366.0, 30.0)
    xg, sg, xo, so = _propagate_both(torch, api, orc, eph, x0, 0.0, t_out)
    assert np.all(sg == 0) and np.all(so == 0)
    err = np.max(np.abs(xg[..., :3] - xo[..., :3]))
    _say(f"sun-only 1 yr max |dx| {err:.3e} au")
    assert err < 1e-10


def test_propagate_j2_enlarged(torch_cuda, orc):
    # Eq. A.4 (App. A.3): an oblate Sun with J2 and radius enlarged so that
    # the term moves close-in bodies far beyond the tolerance, about a
    # tilted pole; the post-Newtonian term on as well
    torch, api = torch_cuda
    rng = np.random.default_rng(31)
    pole = rng.normal(size=3)
    pole /= np.linalg.norm(pole)
    eph = synth.sun_only_ephemeris(-8.0, 45, gr=True, j2=(1e-2, 0.02, pole))
    el = synth.main_belt_elements(rng, 256)
    el[:, 0] = rng.uniform(0.15, 0.8, 256)
    x0 = synth.elements_to_state(*[el[:, k] for k in range(6)], synth.GM_SUN)
    t_out = np.arange(10.0, 340.0, 15.0)
    xg, sg, xo, so = _propagate_both(torch, api, orc, eph, x0, 0.0, t_out)
    assert np.all(sg == 0) and np.all(so == 0)
    err = np.max(np.abs(xg[..., :3] - xo[..., :3]))
    xn, _ = api.propagate(api.DeviceEphemeris.from_synth(synth.sun_only_ephemeris(-8.0, 45, gr=True)),
                          torch.as_tensor(x0).cuda(), 0.0, t_out)
    shift = np.max(np.abs(xn.cpu().numpy()[..., :3] - xg[..., :3]))
    _say(f"enlarged solar J2, 330 d: max |dx| vs oracle {err:.3e} au, J2 shift {shift:.3e} au")
    assert err < 1e-10
    assert shift > 1e-4


def test_propagate_default_model_j2_moon(torch_cuda, orc):
    # the default force model: Sun, planets and the Moon, the Eq. A.3 term
    # for the Sun, Jupiter and the Earth, Eq. A.4 for the Sun and Jupiter;
    # bodies passing close to Jupiter and to the Earth-Moon system
    torch, api = torch_cuda
    model = synth.PlanetModel.make()
    assert model.names[-1] == "moon"
    eph = synth.make_ephemeris(model, -8.0, 50)
    assert eph.j2 is not None and eph.j2[model.names.index("jupiter"), 0] > 0
    rng = np.random.default_rng(32)
    st = model.bary(np.array([100.0]))[0]
    near = []
    # hyperbolic flybys across the offset (closest approach near `dist`),
    # whose straight path keeps clear of the Earth and the Moon
    ie, im = model.names.index("earth"), model.names.index("moon")
    for nm, dist, n, speed in (("jupiter", 0.01, 24, 0.0225), ("earth", 0.003, 24, 5e-3), ("moon", 0.002, 16, 1e-2)):
        b = st[model.names.index(nm)]
        rows = []
        while len(rows) < n:
            off = rng.normal(size=3)
            if nm == "moon":                      # start on the far side from the Earth
                off = 0.3 * off + (b[:3] - st[ie, :3]) / np.linalg.norm(b[:3] - st[ie, :3])
            off *= dist / np.linalg.norm(off)
            dv = np.cross(off, rng.normal(size=3))
            dv *= speed / np.linalg.norm(dv)
            x = np.concatenate([b[:3] + off, b[3:] + dv])
            clear = True
            for k in (ie, im):
                rel, w = x[:3] - st[k, :3], x[3:] - st[k, 3:]
                s = max(0.0, -(rel @ w) / (w @ w))
                clear &= np.linalg.norm(rel + s * w) > 1e-3
            if clear:
                rows.append(x)
        near.append(np.array(rows))
    near = np.concatenate(near)
    far = synth.bodies_from_elements(model, synth.main_belt_elements(rng, 100), 100.0)
    x0 = np.concatenate([near, far])
    t_out = np.arange(103.0, 380.0, 12.0)
    xg, sg, xo, so = _propagate_both(torch, api, orc, eph, x0, 100.0, t_out)
    assert np.all(sg == 0) and np.all(so == 0)
    err = np.max(np.abs(xg[..., :3] - xo[..., :3]))
    _say(f"default model (10 bodies, J2, Moon), flybys of Jupiter, the Earth and the Moon: max |dx| {err:.3e} au")
    assert err < 1e-10


def test_propagate_tiny_config(torch_cuda, orc):
    torch, api = torch_cuda
    case = synth.tiny_case(n_obj=1000, n_frames=100)
    order, off, t_ref = orc.make_batches(case.frames.t)
    xg, sg, xo, so = _propagate_both(torch, api, orc, case.ephem, case.x0, 0.0, t_ref)
    assert np.all(sg == 0) and np.all(so == 0)
    err = np.max(np.abs(xg[..., :3] - xo[..., :3]))
    _say(f"tiny config ({t_ref.size} epochs) max |dx| {err:.3e} au")
    assert err < 1e-10


def test_propagate_survey_mix_one_year(torch_cuda, orc):
    torch, api = torch_cuda
    case = synth.survey_case(n_obj=3000, n_frames=0, neo_frac=0.05)
    t_out = np.arange(1.5, 365.25, 3.0)
    xg, sg, xo, so = _propagate_both(torch, api, orc, case.ephem, case.x0, 0.0, t_out)
    _say(f"survey mix 1 yr: status gpu {np.bincount(sg)}, oracle {np.bincount(so)}")
    np.testing.assert_array_equal(sg, so)
    ok = so == 0
    err = np.abs(xg[..., :3] - xo[..., :3]).max(axis=(0, 2))
    _say(f"survey mix 1 yr: max |dx| {err[ok].max():.3e} au over {ok.sum()} bodies")
    assert ok.all() and err.max() < 1e-10


@pytest.mark.parametrize("n_ast", [4, 7])
def test_propagate_extra_perturbers(torch_cuda, orc, n_ast):
    # Sun + 8 planets + the largest asteroids as extra perturbers: 13
    # bodies, and 16, the most the ABI takes (the run-time body count path)
    torch, api = torch_cuda
    model = synth.PlanetModel.make(synth.PLANET_NAMES + synth.ASTEROID_NAMES[:n_ast], moon=False)
    assert len(model.names) == 9 + n_ast
    eph = synth.make_ephemeris(model, -8.0, 20)
    rng = np.random.default_rng(16 + n_ast)
    x0 = synth.bodies_from_elements(model, np.concatenate([synth.main_belt_elements(rng, 600),
                                                           synth.neo_elements(rng, 30)]), 0.0)
    t_out = np.arange(1.5, 120.0, 3.0)
    xg, sg, xo, so = _propagate_both(torch, api, orc, eph, x0, 0.0, t_out)
    ok = (sg == 0) & (so == 0)
    assert ok.all()
    err = np.abs(xg[..., :3] - xo[..., :3]).max()
    # the asteroids move the bodies measurably against the planets alone
    xp, _ = api.propagate(api.DeviceEphemeris.from_synth(
        synth.make_ephemeris(synth.PlanetModel.make(moon=False), -8.0, 20)), _dev_x(torch, x0), 0.0, t_out)
    shift = np.abs(xp.cpu().numpy()[..., :3] - xg[..., :3]).max()
    _say(f"{len(model.names)} perturbers, 120 d: max |dx| vs oracle {err:.3e} au, shift from the asteroids "
         f"{shift:.3e} au")
    assert err < 1e-10
    assert shift > 1e-11


def test_propagate_backward(torch_cuda, orc):
    torch, api = torch_cuda
    model = synth.PlanetModel.make()
    e = synth.make_ephemeris(model, -216.0, 40)
    rng = np.random.default_rng(14)
    x0, _, _ = synth.make_population(rng, model, 500, 0.1, 0.0)
    t_out = np.array([-3.0, -50.0, -120.5, -200.0])
    xg, sg, xo, so = _propagate_both(torch, api, orc, e, x0, 0.0, t_out)
    assert np.all(sg == 0) and np.all(so == 0)
    err = np.max(np.abs(xg[..., :3] - xo[..., :3]))
    _say(f"backward 200 d max |dx| {err:.3e} au")
    assert err < 1e-10


def test_propagate_configuration_invariance(torch_cuda):
    torch, api = torch_cuda
    case = synth.survey_case(n_obj=777, n_frames=0, neo_frac=0.2)
    eph = api.DeviceEphemeris.from_synth(case.ephem)
    x0 = _dev_x(torch, case.x0)
    t_out = np.arange(3.0, 100.0, 3.0)
    ref, st = api.propagate(eph, x0, 0.0, t_out, api.default_opts())
    ref2, _ = api.propagate(eph, x0, 0.0, t_out, api.default_opts())
    assert torch.equal(ref, ref2), "propagation is not deterministic"
    for kw in (dict(n_buckets=1), dict(block=64), dict(block=128, n_buckets=4), dict(rebucket_epochs=1),
               dict(window_segs=1), dict(rebucket_epochs=0), dict(rebucket_epochs=16), dict(lanes_per_body=7),
               dict(lanes_per_body=8), dict(lanes_per_body=7, block=256), dict(lanes_per_body=1),
               dict(zero_start=1), dict(zero_start=1, lanes_per_body=8)):
        x, s = api.propagate(eph, x0, 0.0, t_out, api.default_opts(**kw))
        d = (x - ref).abs().max().item()
        _say(f"config {kw}: max |dx| vs default {d:.3e}")
        assert d < 1e-11
        assert torch.equal(s, st)


def test_extrapolated_corrector_start(torch_cuda, orc):
    """The grouped integrators start each corrector from the previous
    step's increments extrapolated: nearly every step after the first is
    counted as predicted, the corrector needs fewer sweeps than from zero,
    and both starts agree with the oracle (which starts from zero)."""
    torch, api = torch_cuda
    case = synth.survey_case(n_obj=600, n_frames=0, neo_frac=0.2)
    eph = api.DeviceEphemeris.from_synth(case.ephem)
    x0 = _dev_x(torch, case.x0)
    t_out = np.arange(3.0, 121.0, 3.0)
    xp, sp, stp = api.propagate(eph, x0, 0.0, t_out, api.default_opts(), stats=True)
    xz, sz, stz = api.propagate(eph, x0, 0.0, t_out, api.default_opts(zero_start=1), stats=True)
    stp, stz = stp.cpu().numpy(), stz.cpu().numpy()
    sweeps_p, sweeps_z = stp[4] / stp[3], stz[4] / stz[3]
    _say(f"sweeps per body-step: extrapolated start {sweeps_p:.2f}, zero start {sweeps_z:.2f}; "
         f"predicted steps {stp[7] / stp[3]:.3f}")
    assert stz[7] == 0
    assert stp[7] > 0.9 * stp[3]
    assert sweeps_p < 0.8 * sweeps_z
    assert torch.equal(sp, sz)
    sel = np.arange(0, 600, 25)
    xo, so, _ = orc.propagate(case.ephem, case.x0[sel], 0.0, t_out)
    for x in (xp, xz):
        xs = x[:, torch.as_tensor(sel, device="cuda")].cpu().numpy()
        assert np.max(np.abs(xs[..., :3] - xo[..., :3])) < 1e-10


def test_dense_epochs_match_landing(torch_cuda, orc):
    """Epochs read off the step polynomials (the default) against landing on
    every epoch and against the oracle, which lands: an epoch equal to the
    start, epochs a fraction of a step apart, backward integration and runs
    split over several launches."""
    torch, api = torch_cuda
    case = synth.survey_case(n_obj=300, n_frames=0, neo_frac=0.2)
    eph = api.DeviceEphemeris.from_synth(case.ephem)
    x0 = _dev_x(torch, case.x0)
    sel = np.arange(0, 300, 7)
    for t0, t_out in ((0.0, [0.0, 0.7, 3.1, 3.2, 10.0, 17.5, 40.0, 61.25]), (30.0, [29.5, 21.0, 20.9, 2.0])):
        xd, sd, std = api.propagate(eph, x0, t0, t_out, api.default_opts(), stats=True)
        xl, sl, stl = api.propagate(eph, x0, t0, t_out, api.default_opts(land_epochs=1), stats=True)
        xr, sr = api.propagate(eph, x0, t0, t_out, api.default_opts(rebucket_epochs=3))
        assert torch.equal(sd, sl) and torch.equal(sd, sr)
        ok = (sd == 0).cpu().numpy()
        d_land = (xd - xl)[:, torch.as_tensor(ok, device="cuda")].abs().max().item()
        d_split = (xd - xr)[:, torch.as_tensor(ok, device="cuda")].abs().max().item()
        xo, so, _ = orc.propagate(case.ephem, case.x0[sel], t0, t_out)
        xs = xd[:, torch.as_tensor(sel, device="cuda")].cpu().numpy()
        d_orc = np.abs(xs[:, so == 0, :3] - xo[:, so == 0, :3]).max()
        _say(f"t0 {t0}: dense vs landing {d_land:.2e}, vs split launches {d_split:.2e}, vs oracle {d_orc:.2e} au; "
             f"body-steps {std.cpu().numpy()[3]} vs {stl.cpu().numpy()[3]} landing")
        assert d_land < 1e-11 and d_split < 1e-11 and d_orc < 1e-11
        assert std.cpu().numpy()[3] < stl.cpu().numpy()[3]
        # the epoch at the start time is the initial state itself
        if t_out[0] == t0:
            assert torch.equal(xd[0], x0)


def test_propagate_ragged_sizes(torch_cuda, orc):
    torch, api = torch_cuda
    case = synth.survey_case(n_obj=130, n_frames=0, neo_frac=0.3)
    t_out = [2.0, 9.5]
    for lanes in (7, 8, 1):
        for n in (1, 8, 9, 10, 17, 63, 65, 130):
            xg, sg, xo, so = _propagate_both(torch, api, orc, case.ephem, case.x0[:n], 0.0, t_out,
                                             lanes_per_body=lanes)
            assert np.max(np.abs(xg - xo)) < 1e-12, (lanes, n)
    eph = api.DeviceEphemeris.from_synth(case.ephem)
    x, s = api.propagate(eph, torch.zeros((0, 6), dtype=torch.float64, device="cuda"), 0.0, t_out)
    assert x.shape == (2, 0, 6)


def test_propagate_status_codes(torch_cuda, orc):
    torch, api = torch_cuda
    case = synth.survey_case(n_obj=200, n_frames=0)
    x0 = case.x0.copy()
    x0[7] = np.nan
    eph = api.DeviceEphemeris.from_synth(case.ephem)
    x, s = api.propagate(eph, _dev_x(torch, x0), 0.0, [10.0, 20.0])
    s = s.cpu().numpy(); x = x.cpu().numpy()
    assert s[7] == 1 and np.all(np.isnan(x[:, 7]))
    good = np.arange(200) != 7
    assert np.all(s[good] == 0)
    xo, so, _ = orc.propagate(case.ephem, case.x0[good], 0.0, [10.0, 20.0])
    assert np.max(np.abs(x[:, good] - xo)) < 1e-12
    _, s2 = api.propagate(eph, _dev_x(torch, case.x0), 0.0, [300.0], api.default_opts(max_steps=3))
    assert np.all(s2.cpu().numpy() == 3)
    _, s3 = api.propagate(eph, _dev_x(torch, case.x0), 0.0, [300.0], api.default_opts(h_min=200.0))
    assert np.all(s3.cpu().numpy() == 2)


@pytest.mark.parametrize("n,span", [(1, 220.0), (2048, 220.0), (2049, 220.0), (8193, 220.0), (9217, 220.0),
                                    (220000, 20.0)])
def test_lone_paired_and_grouped_objects(torch_cuda, n, span):
    """The list sizes at which objects move between wavefronts of their own,
    two lanes per node and nine a wavefront, against the 8-lane groups: with
    fast orbits of many steps among them, more epochs inside a step and in
    all than a wavefront's lanes hold, and none of the last launch's state."""
    torch, api = torch_cuda
    case = synth.survey_case(n_obj=n, n_frames=0, neo_frac=0.3)
    eph = api.DeviceEphemeris.from_synth(case.ephem)
    x0 = _dev_x(torch, case.x0)
    t_out = np.concatenate([np.linspace(0.0, 12.0, 70 if n < 100000 else 3), [span]])
    for back in (False, True):
        t0, t = (span, span - t_out) if back else (0.0, t_out)
        x, s = api.propagate(eph, x0, t0, t)
        y, r = api.propagate(eph, x0, t0, t, api.default_opts(lanes_per_body=8))
        assert torch.equal(s, r) and int(s.abs().max()) == 0
        d = (x - y).abs().max().item()
        _say(f"n {n} back {back}: max |dx| vs 8-lane groups {d:.3e}")
        assert d < 1e-10


def test_shared_wavefronts_line_up_perihelion_passages(torch_cuda):
    """Fast orbits that share wavefronts (eight lanes or one a body) pass
    perihelion together: they take fewer shared steps than in the order of
    their numbers of steps, in which each shortens the others' steps at times
    of its own."""
    torch, api = torch_cuda
    rng = np.random.default_rng(95)
    model = synth.PlanetModel.make()
    eph = api.DeviceEphemeris.from_synth(synth.make_ephemeris(model, -8.0, 49))
    el = synth.neo_elements(rng, 8000)
    el = el[el[:, 0] < 1.0]                              # a passage or more a year
    x = synth.bodies_from_elements(model, el, 0.0)
    q = el[:, 0] * (1 - el[:, 1])
    by_steps = np.argsort(q ** 1.5 / np.sqrt(1 + el[:, 1]))      # the predicted step at perihelion
    steps = {}
    for lanes in (8, 1):
        for name, order, buckets in (("own", np.arange(len(x)), 16), ("by steps", by_steps, 1)):
            opts = api.default_opts(lanes_per_body=lanes, n_buckets=buckets)
            _, st, c = api.propagate(eph, _dev_x(torch, x[order]), 0.0, [365.0], opts, stats=True)
            assert int(st.abs().max()) == 0
            steps[lanes, name] = int(c[0])
    _say(f"{len(x)} bodies, shared steps {steps}")
    for lanes in (8, 1):
        assert steps[lanes, "own"] < 0.97 * steps[lanes, "by steps"]


@pytest.mark.parametrize("n,n_out", [(2049, 5), (9300, 3), (9300, 4), (9300, 70)])
def test_many_epochs_of_a_day(torch_cuda, n, n_out):
    """Objects that cross the span in one step keep their order when their
    epochs are many; the states are those of the unsorted run."""
    torch, api = torch_cuda
    case = synth.survey_case(n_obj=n, n_frames=0, neo_frac=0.3)
    eph = api.DeviceEphemeris.from_synth(case.ephem)
    x0 = _dev_x(torch, case.x0)
    for end in (1.0, -1.0, 4.0):
        t_out = np.linspace(0.0, end, n_out + 1)[1:]
        x, s = api.propagate(eph, x0, 0.0, t_out)
        y, r = api.propagate(eph, x0, 0.0, t_out, api.default_opts(n_buckets=1))
        assert torch.equal(s, r) and int(s.abs().max()) == 0
        assert (x - y).abs().max().item() < 1e-12


@pytest.mark.parametrize("n", [40, 3000, 9300])
@pytest.mark.parametrize("table", ["degree 9", "J2 without Eq. A.3", "four bodies", "no J2", "no Eq. A.3"])
def test_propagate_other_tables(torch_cuda, table, n):
    """Perturber tables that the unrolled force does not cover, in each of
    the wavefront layouts, against the one-lane integrator."""
    torch, api = torch_cuda
    case = synth.survey_case(n_obj=n, n_frames=0, neo_frac=0.2)
    e = case.ephem
    flags, j2 = e.flags.copy(), e.j2.copy()
    bodies = list(range(e.n_body))
    if table == "J2 without Eq. A.3": flags[np.nonzero(j2[:, 0])[0][-1]] = 0
    if table == "four bodies": bodies = bodies[:4]
    if table == "no J2": j2[:] = 0.0
    if table == "no Eq. A.3": flags[:] = 0
    coef = e.coef[bodies][..., :10] if table == "degree 9" else e.coef[bodies]
    e = dataclasses.replace(e, coef=np.ascontiguousarray(coef), gm=e.gm[bodies], flags=flags[bodies],
                            names=[e.names[b] for b in bodies], j2=np.ascontiguousarray(j2[bodies]))
    eph = api.DeviceEphemeris.from_synth(e)
    x0 = _dev_x(torch, case.x0)
    t_out = [1.0, 30.0, 60.0]
    x, s = api.propagate(eph, x0, 0.0, t_out)
    y, r = api.propagate(eph, x0, 0.0, t_out, api.default_opts(lanes_per_body=1))
    assert torch.equal(s, r) and int(s.abs().max()) == 0
    d = (x - y).abs().max().item()
    _say(f"{table}, n {n}: max |dx| vs one lane per object {d:.3e}")
    assert d < 1e-11


@pytest.mark.parametrize("bodies,n_seg", [(10, 6_200_000), (2, 2 ** 32 // 39 + 2)])
def test_ephemeris_table_past_2_31_values(torch_cuda, bodies, n_seg):
    """The same segments in a table so long that the last bodies' lie past
    2^31 values (19 GB) and even one body has 2^32 (69 GB): the same states and
    gradients, the latter's up to the rounding of another kernel shape."""
    torch, api = torch_cuda
    torch.cuda.empty_cache()
    case = synth.survey_case(n_obj=2100, n_frames=0)
    e = case.ephem
    e = dataclasses.replace(e, coef=e.coef[:bodies], gm=e.gm[:bodies], flags=e.flags[:bodies], names=e.names[:bodies],
                            j2=e.j2[:bodies])
    eph, far = (api.DeviceEphemeris.from_synth(e) for _ in range(2))
    nb, ns, _, m = eph.coef.shape
    assert (nb - 1) * n_seg * 3 * m > 2 ** 31
    tol = 0.0 if bodies == 10 else 1e-13
    if torch.cuda.mem_get_info()[0] < 10 * nb * n_seg * 3 * m:
        pytest.skip("not enough free device memory")
    far.coef = torch.zeros((nb, n_seg, 3, m), dtype=torch.float64, device="cuda")
    far.coef[:, :ns] = eph.coef
    far.c.n_seg, far.c.coef = n_seg, far.coef.data_ptr()
    x0 = _dev_x(torch, case.x0)
    for n, lanes in ((40, 7), (2100, 7), (40, 8), (40, 1)):
        o = api.default_opts(lanes_per_body=lanes)
        x, s = api.propagate(eph, x0[:n], 0.0, [5.0, 30.0], o)
        y, r = api.propagate(far, x0[:n], 0.0, [5.0, 30.0], o)
        assert torch.equal(s, r) and (x - y).abs().max().item() <= tol, (n, lanes)
    t_obs = _dev_x(torch, np.tile([3.0, 9.0, 20.0], (40, 1)))
    grads = []
    for e in (eph, far):
        ctx = api.AdjointContext(e, 0.0, 20.0, t_obs, _dev_x(torch, np.tile([1.0, 0.1, 0.0], (40, 3, 1))))
        sky = ctx.forward(x0[:40])
        grads.append((sky, ctx.backward(x0[:40], torch.ones_like(sky))))
    for a, b in zip(*grads):
        assert (a - b).abs().max().item() <= 1e3 * tol * b.abs().max().item()
    del far
    torch.cuda.empty_cache()


@pytest.mark.parametrize("n", [1, 8, 9, 200])
@pytest.mark.parametrize("lanes", [0, 1, 7, 8])
def test_propagate_all_objects_of_a_wavefront_fail(torch_cuda, n, lanes):
    """Every epoch after the failure is NaN, also those that the integrator
    would have passed inside a step, where no object of a wavefront is left."""
    torch, api = torch_cuda
    case = synth.survey_case(n_obj=n, n_frames=0)
    eph = api.DeviceEphemeris.from_synth(case.ephem)
    epochs = [0.0, 2.0, 5.0, 9.0, 40.0]
    opts = api.default_opts(lanes_per_body=lanes) if lanes else api.default_opts()
    x, s = api.propagate(eph, _dev_x(torch, case.x0), 0.0, epochs, opts)
    assert np.all(s.cpu().numpy() == 0) and np.all(np.isfinite(x.cpu().numpy()))
    del x, s                        # the next outputs take the same memory
    opts.h_min = 200.0
    x, s = api.propagate(eph, _dev_x(torch, case.x0), 0.0, epochs, opts)
    x = x.cpu().numpy()
    assert np.all(s.cpu().numpy() == 2)
    assert np.array_equal(x[0], case.x0) and np.all(np.isnan(x[1:]))


@pytest.mark.parametrize("n", [9, 3000])
def test_epochs_close_to_the_last_one(torch_cuda, n):
    """Epochs a few ulps before the one that a launch lands on, which is
    reached by a step across t = 0: start + (end - start) may round below
    them, and their states are those of the end all the same."""
    torch, api = torch_cuda
    case = synth.survey_case(n_obj=n, n_frames=0)
    eph = api.DeviceEphemeris.from_synth(case.ephem)
    x0 = _dev_x(torch, case.x0)
    rng = np.random.default_rng(92)
    below = 0
    for _ in range(20):
        t0, end = rng.uniform(-7.5, -1.0), rng.uniform(0.1, 3.0)
        t_out = end - np.spacing(end) * np.arange(40, -1, -1)
        below += t0 + (end - t0) < t_out[-2]
        for lanes in (7, 8):
            x, s = api.propagate(eph, x0, t0, t_out, api.default_opts(lanes_per_body=lanes))
            assert int(s.abs().max()) == 0
            assert (x - x[-1]).abs().max().item() < 1e-13, (t0, end, lanes)
    assert below > 0


# ---------------------------------------------------------------- FoV
def _pair_set(pf, ps, po):
    return set(zip(np.asarray(pf).tolist(), np.asarray(ps).tolist(), np.asarray(po).tolist()))


def _compare_pairs(gpu, orc_pairs, edge, label):
    g = _pair_set(*gpu)
    o = _pair_set(*orc_pairs)
    near = {k for k, e in zip(zip(*[np.asarray(a).tolist() for a in orc_pairs]), edge) if abs(e) < MAS}
    missing = o - g - near
    extra = g - o
    _say(f"{label}: oracle {len(o)} pairs, gpu {len(g)}, missing {len(missing)}, extra {len(extra)}")
    assert not missing, sorted(missing)[:10]
    # an extra GPU pair must sit within 1 mas of an edge of its frame
    return extra


def _edge_of(orc, ephem, x_epoch, order, off, t_ref, fr, pair):
    f, s, j = pair
    q = int(np.nonzero(order == f)[0][0])
    b = int(np.searchsorted(off, q, side="right") - 1)
    st, d, tau, _ = orc.lighttime(ephem, t_ref[b], x_epoch[b, j], fr.t[f], fr.obs[f])
    ins, edge = orc.inside(fr.normals[f], d)
    return edge[s]


def _fov_case(torch, api, orc, case, x_epoch_host, order, off, t_ref, opts=None, status=None):
    eph = api.DeviceEphemeris.from_synth(case.ephem)
    fr = api.DeviceFrames.from_synth(case.frames)
    b = api.Batches.from_host(order.astype(np.int32), off.astype(np.int32), t_ref)
    pf, ps, po, stats = api.fov_check(eph, _dev_x(torch, x_epoch_host), b, fr, status, opts, return_stats=True)
    _say(f"fov stats (candidates, exact, brute-force objects): {stats[:3].tolist()}")
    return pf.cpu().numpy(), ps.cpu().numpy(), po.cpu().numpy()


def test_fov_given_oracle_states(torch_cuda, orc):
    torch, api = torch_cuda
    case = synth.tiny_case(n_obj=1000, n_frames=100, n_targeted=400)
    fr = case.frames
    order, off, t_ref = orc.make_batches(fr.t)
    xe, st, _ = orc.propagate(case.ephem, case.x0, 0.0, t_ref)
    opairs = orc.fov(case.ephem, xe, st, order, off, t_ref, fr.t, fr.obs, fr.normals)
    gp = _fov_case(torch, api, orc, case, xe, order, off, t_ref)
    assert np.all(np.diff(gp[0].astype(np.int64) * 2 ** 32 + gp[1].astype(np.int64) * 2 ** 25 + gp[2]) > 0)
    extra = _compare_pairs(gp, opairs[:3], opairs[3], "tiny+targeted given oracle states")
    for p in extra:
        assert abs(_edge_of(orc, case.ephem, xe, order, off, t_ref, fr, p)) < MAS
    assert len(opairs[0]) > 200


def test_fov_distant_bodies(torch_cuda, orc):
    """Bodies from 30 au to 400 au (light times up to 2.3 days, where the
    exact test's Sun cubic is re-expanded about each body's emission time)
    among main-belt bodies, with frames aimed at them: the pair sets must
    match the oracle's."""
    torch, api = torch_cuda
    case = synth.tiny_case(n_obj=600, n_frames=40)
    rng = np.random.default_rng(16)
    n_far = 240
    a = np.concatenate([rng.uniform(30.0, 60.0, n_far - 40), rng.uniform(150.0, 400.0, 40)])
    e = rng.uniform(0.0, 0.2, n_far)
    inc = rng.rayleigh(math.radians(10.0), n_far)
    ang = rng.uniform(0.0, 2.0 * np.pi, (3, n_far))
    el_far = np.stack([a, e, inc, ang[0], ang[1], ang[2]], axis=1)
    x_far = synth.bodies_from_elements(case.model, el_far, 0.0)
    x0 = np.concatenate([case.x0, x_far])
    fr = synth.Frames.concat([case.frames, synth.frames_targeted(rng, case.model, el_far, 0.0, case.span, 160)])
    fr = fr.subset(np.argsort(fr.t, kind="stable"))
    case = synth.PropagationCase("tiny-far", case.ephem, case.model, x0, None, np.zeros(x0.shape[0], bool), 0.0,
                                 case.span, fr, 16)
    order, off, t_ref = orc.make_batches(fr.t)
    xe, st, _ = orc.propagate(case.ephem, x0, 0.0, t_ref)
    opairs = orc.fov(case.ephem, xe, st, order, off, t_ref, fr.t, fr.obs, fr.normals)
    gp = _fov_case(torch, api, orc, case, xe, order, off, t_ref)
    extra = _compare_pairs(gp, opairs[:3], opairs[3], "distant bodies given oracle states")
    for p in extra:
        assert abs(_edge_of(orc, case.ephem, xe, order, off, t_ref, fr, p)) < MAS
    far_pairs = int(np.sum(np.asarray(opairs[2]) >= 600))
    _say(f"pairs of the distant bodies: {far_pairs}")
    assert far_pairs > 100


def test_fov_full_chain_tiny(torch_cuda, orc):
    torch, api = torch_cuda
    case = synth.tiny_case(n_obj=1000, n_frames=100, n_targeted=300)
    fr = case.frames
    eph = api.DeviceEphemeris.from_synth(case.ephem)
    pf, ps, po, xg, sg, bt = api.predict(eph, _dev_x(torch, case.x0), 0.0, api.DeviceFrames.from_synth(fr), fr.t)
    order, off, t_ref = orc.make_batches(fr.t)
    np.testing.assert_array_equal(bt.t_ref_host, t_ref)
    xe, st, _ = orc.propagate(case.ephem, case.x0, 0.0, t_ref)
    assert np.max(np.abs(xg.cpu().numpy() - xe)) < 1e-10
    opairs = orc.fov(case.ephem, xe, st, order, off, t_ref, fr.t, fr.obs, fr.normals)
    extra = _compare_pairs((pf.cpu().numpy(), ps.cpu().numpy(), po.cpu().numpy()), opairs[:3], opairs[3],
                           "tiny full chain")
    for p in extra:
        assert abs(_edge_of(orc, case.ephem, xe, order, off, t_ref, fr, p)) < MAS


def test_fov_survey_geometry(torch_cuda, orc):
    torch, api = torch_cuda
    case = synth.survey_case(n_obj=20000, n_frames=20000, span=20.0, neo_frac=0.05)
    fr = case.frames
    order, off, t_ref = orc.make_batches(fr.t)
    eph = api.DeviceEphemeris.from_synth(case.ephem)
    xg, sg = api.propagate(eph, _dev_x(torch, case.x0), 0.0, t_ref)
    b = api.Batches.from_host(order.astype(np.int32), off.astype(np.int32), t_ref)
    pf, ps, po, stats = api.fov_check(eph, xg, b, api.DeviceFrames.from_synth(fr), sg, return_stats=True)
    _say(f"survey geometry stats {stats.tolist()}, pairs {pf.numel()}")
    # oracle on a sample of objects, all frames
    rng = np.random.default_rng(15)
    sample = np.sort(rng.choice(case.x0.shape[0], 600, replace=False))
    xe, st, _ = orc.propagate(case.ephem, case.x0[sample], 0.0, t_ref)
    opf, ops, opo, oedge = orc.fov(case.ephem, xe, st, order, off, t_ref, fr.t, fr.obs, fr.normals)
    opo = sample[opo]
    keep = np.isin(po.cpu().numpy(), sample)
    gp = (pf.cpu().numpy()[keep], ps.cpu().numpy()[keep], po.cpu().numpy()[keep])
    extra = _compare_pairs(gp, (opf, ops, opo), oedge, "survey geometry sample")
    # an extra GPU pair lies within 1 mas of an edge, measured from the oracle's states
    loc = {int(j): i for i, j in enumerate(sample)}
    for f, s, j in extra:
        assert abs(_edge_of(orc, case.ephem, xe, order, off, t_ref, fr, (f, s, loc[j]))) < MAS, (f, s, j)


@pytest.mark.parametrize("n_obj", [1, 63, 64, 65, 3000])
@pytest.mark.parametrize("n_sub", [1, 16, 64, 120])
def test_fov_few_frames_a_batch(torch_cuda, n_sub, n_obj):
    """Batches of few frames, which are joined without a sky grid, give the
    pairs that the sorted join finds: the same frames three times over are
    enough of them for that one.  No frames, one, and more than a wavefront's
    share to a batch; among the objects a failed one, one without a state,
    one at the observer and one too fast for a bound."""
    torch, api = torch_cuda
    sizes = [1, 0, 5, 64, 65, 130]
    case = synth.footprint_case(n_obj=3000, n_frames=sum(sizes), span=12.0)
    fr = case.frames
    if n_sub == 1: fr = dataclasses.replace(fr, normals=np.ascontiguousarray(fr.normals[:, :1]))
    if n_sub in (16, 120): fr = _random_layout_frames(np.random.default_rng(83), fr, n_sub=n_sub)
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    order = np.argsort(fr.t, kind="stable").astype(np.int32)
    ts = fr.t[order]
    t_ref = np.array([0.5 * (ts[a] + ts[b - 1]) if b > a else 0.5 * (ts[a - 1] + ts[a])
                      for a, b in zip(off[:-1], off[1:])])
    eph = api.DeviceEphemeris.from_synth(case.ephem)
    x, st = api.propagate(eph, _dev_x(torch, case.x0[:n_obj]), 0.0, t_ref)
    if n_obj > 60:
        st[3] = 1
        x[5, 7] = float("nan")
        x[4, 9, :3] = torch.as_tensor(fr.obs[order[off[4]]], device="cuda")
        x[3, 11, 3:] = 100.0
    b1 = api.Batches.from_host(order, off, t_ref)
    F, R = fr.t.size, 3
    # copy c of frame f is frame c F + f, in the same batch
    order3 = np.concatenate([(order[a:b, None] + F * np.arange(R)).ravel() for a, b in zip(off[:-1], off[1:])])
    b3 = api.Batches.from_host(order3.astype(np.int32), R * off, t_ref)
    fr3 = dataclasses.replace(fr, t=np.tile(fr.t, R), obs=np.tile(fr.obs, (R, 1)),
                              normals=np.tile(fr.normals, (R, 1, 1, 1)))
    s1, s3 = st.clone(), st.clone()
    pf, ps, po, c1 = api.fov_check(eph, x, b1, api.DeviceFrames.from_synth(fr), s1, return_stats=True)
    qf, qs, qo, c3 = api.fov_check(eph, x, b3, api.DeviceFrames.from_synth(fr3), s3, return_stats=True)
    _say(f"n_obj {n_obj}, n_sub {n_sub}: {pf.numel()} pairs, stats {c1.tolist()} against {c3.tolist()}")
    assert torch.equal(s1, s3)
    assert n_obj < 3000 or pf.numel() > 0
    # both lists are sorted by (frame, sub-frame, object): the copies follow each other
    assert torch.equal(qf, torch.cat([pf + c * F for c in range(R)]).to(qf.dtype))
    assert torch.equal(qs, ps.repeat(R)) and torch.equal(qo, po.repeat(R))


@pytest.mark.parametrize("n_sub", [1, 64])
def test_fov_frames_outside_every_batch(torch_cuda, n_sub):
    """Ranks before the first batch's and behind the last one's are tested
    with those batches, whichever join a call's numbers choose (here the same
    frames once and three times over).  They hold copies of frames of those
    batches, whose bounds so cover them."""
    torch, api = torch_cuda
    case = synth.footprint_case(n_obj=3000, n_frames=90, span=5.0)
    fr = case.frames
    if n_sub == 1: fr = dataclasses.replace(fr, normals=np.ascontiguousarray(fr.normals[:, :1]))
    order = np.argsort(fr.t, kind="stable")
    order = np.concatenate([order[[10, 20, 30]], order, order[[50, 55, 60, 65, 70, 75, 87]]])
    fr = dataclasses.replace(fr, t=fr.t[order], obs=fr.obs[order], normals=fr.normals[order])
    t_ref = np.array([fr.t[3:43].mean(), fr.t[43:93].mean()])
    eph = api.DeviceEphemeris.from_synth(case.ephem)
    x, _ = api.propagate(eph, _dev_x(torch, case.x0), 0.0, t_ref)
    for copies in (1, 3):
        some = dataclasses.replace(fr, t=fr.t.repeat(copies), obs=fr.obs.repeat(copies, axis=0),
                                   normals=fr.normals.repeat(copies, axis=0))
        frames = api.DeviceFrames.from_synth(some)
        pairs = []
        for off in ([0, 43, 100], [3, 43, 93]):
            b = api.Batches.from_host(np.arange(100 * copies, dtype=np.int32),
                                      np.array(off, np.int32) * copies, t_ref)
            pairs.append(api.fov_check(eph, x, b, frames))
        _say(f"n_sub {n_sub}, {copies} of each: {pairs[0][0].numel()} pairs, "
             f"{int((pairs[0][0] < 3 * copies).sum() + (pairs[0][0] >= 93 * copies).sum())} of them outside")
        assert int((pairs[0][0] < 3 * copies).sum()) > 0 and int((pairs[0][0] >= 93 * copies).sum()) > 0
        for a, c in zip(*pairs):
            assert torch.equal(a, c)


@pytest.mark.parametrize("widest", [165.0, 180.0])
def test_fov_sub_frames_far_apart(torch_cuda, orc, widest):
    """Frames of two sub-frames 10 degrees apart and more, 120 to a batch.  Up
    to 165 degrees, boxes that reach tangents of 12 about the frame's centre,
    in the per-cell join; up to 180, frames without a box (a vertex outside
    the centre's hemisphere), whose batch's bodies all take the wide join.
    Every pair is the oracle's."""
    torch, api = torch_cuda
    rng = np.random.default_rng(96)
    base = synth.tiny_case(n_obj=1500, n_frames=1, span=6.0)
    F = 240
    t = np.sort(rng.uniform(0.2, 5.8, F))
    obs = synth.circular_observer(base.model, t)[:, :3]
    lon, lat = rng.uniform(0, 2 * np.pi, F), rng.uniform(-0.1, 0.1, F)
    sep = np.radians(np.resize(np.array([10.0, 60.0, 120.0, 150.0, 170.0, 175.0, 178.0, 180.0]) * (widest / 180.0), F))
    subs = []
    for a in (-0.5, 0.5):
        c = np.stack([np.cos(lon + a * sep) * np.cos(lat), np.sin(lon + a * sep) * np.cos(lat), np.sin(lat)], axis=1)
        h = np.full(F, np.radians(2.0))
        subs.append(synth.rect_normals(c, *synth.tangent_basis(c), h, h))
    fr = synth.Frames(t, obs, None, None, None, None, None, np.stack(subs, axis=1))
    case = dataclasses.replace(base, frames=fr)
    order, off, t_ref = orc.make_batches(t)
    assert F > 96 * (len(off) - 1)
    xe, st, _ = orc.propagate(case.ephem, case.x0, 0.0, t_ref)
    opairs = orc.fov(case.ephem, xe, st, order, off, t_ref, t, obs, fr.normals)
    *gp, stats = api.fov_check(api.DeviceEphemeris.from_synth(case.ephem), _dev_x(torch, xe),
                               api.Batches.from_host(order.astype(np.int32), off.astype(np.int32), t_ref),
                               api.DeviceFrames.from_synth(fr), return_stats=True)
    gp = [a.cpu().numpy() for a in gp]
    found = np.bincount(np.arange(F)[opairs[0]] % 8, minlength=8)
    _say(f"{len(opairs[0])} pairs, by separation {found.tolist()}; {stats[2]} of 3000 without a bound")
    assert found.min() > 0
    assert stats[2] == 3000 if widest == 180.0 else stats[2] < 300
    extra = _compare_pairs(gp, opairs[:3], opairs[3], "sub-frames far apart")
    for p in extra:
        assert abs(_edge_of(orc, case.ephem, xe, order, off, t_ref, fr, p)) < MAS


@pytest.mark.parametrize("copies", [1, 31, 32, 33, 1023, 1025, 4097, 8193])
def test_fov_pairs_of_a_frame_sorted(torch_cuda, copies):
    """Copies of one object, as many pairs in each frame that holds it: the
    sizes at which the sort of a frame's pairs changes hands."""
    torch, api = torch_cuda
    case = synth.footprint_case(n_obj=1500, n_frames=300, span=3.0)
    eph = api.DeviceEphemeris.from_synth(case.ephem)
    fr = api.DeviceFrames.from_synth(case.frames)
    order, off, t_ref = api.make_batches(case.frames.t, 3.0)
    x, _ = api.propagate(eph, _dev_x(torch, case.x0), 0.0, t_ref)
    b = api.Batches.from_host(order, off, t_ref)
    pf, ps, po = api.fov_check(eph, x, b, fr)
    j = int(torch.bincount(po.long()).argmax())           # the object of most pairs
    one = torch.nonzero(po == j)[:, 0]
    f1, s1 = pf[one], ps[one]
    qf, qs, qo = api.fov_check(eph, x[:, j:j + 1].expand(-1, copies, -1).contiguous(), b, fr)
    assert torch.equal(qf, f1.repeat_interleave(copies))
    assert torch.equal(qs, s1.repeat_interleave(copies))
    assert torch.equal(qo, torch.arange(copies, device="cuda", dtype=qo.dtype).repeat(one.numel()))


@pytest.mark.parametrize("n_frames", [8191, 8192, 8193, (1 << 20) + 1])
def test_fov_frame_counts(torch_cuda, n_frames):
    """Numbers of frames at which the prefix sums over them change hands:
    copies of 300 frames, each with its original's pairs."""
    torch, api = torch_cuda
    case = synth.footprint_case(n_obj=5000, n_frames=300, span=3.0)
    fr = dataclasses.replace(case.frames, normals=np.ascontiguousarray(case.frames.normals[:, 20:21]))
    eph = api.DeviceEphemeris.from_synth(case.ephem)
    x, _ = api.propagate(eph, _dev_x(torch, case.x0), 0.0, [1.5])
    one = lambda n: api.Batches.from_host(np.arange(n, dtype=np.int32), np.array([0, n], np.int32), np.array([1.5]))
    pf, ps, po = api.fov_check(eph, x, one(300), api.DeviceFrames.from_synth(fr))
    assert pf.numel() > 0
    k = np.arange(n_frames) % 300
    many = dataclasses.replace(fr, t=fr.t[k], obs=fr.obs[k], normals=fr.normals[k])
    qf, qs, qo = api.fov_check(eph, x, one(n_frames), api.DeviceFrames.from_synth(many))
    c = torch.arange((n_frames + 299) // 300, device="cuda")[:, None] * 300
    f = (c + pf[None, :].long()).ravel()
    keep = f < n_frames
    assert torch.equal(qf.long(), f[keep])
    assert torch.equal(qo, po.repeat(c.shape[0])[keep]) and int(qs.abs().max()) == 0


@pytest.mark.parametrize("n_frames", [1 << 27, (1 << 28) + 3])
def test_fov_very_many_frames(torch_cuda, n_frames):
    """As many frames as pass the threads of one launch with 32 a frame, and
    as many as pass 32 bits with eight values a frame (some 700 bytes a frame,
    inputs and workspace): all away from the one body but a handful that hold
    it."""
    torch, api = torch_cuda
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < 760 * n_frames:
        pytest.skip("not enough free device memory")
    case = synth.footprint_case(n_obj=1, n_frames=0, span=3.0)
    eph = api.DeviceEphemeris.from_synth(case.ephem)
    x, _ = api.propagate(eph, _dev_x(torch, case.x0), 0.0, [1.5])
    obs = np.array([1.0, 0.1, 0.0])
    d, _ = api.lighttime_directions(eph, x[0], 1.5, _dev_x(torch, [1.5]), _dev_x(torch, obs[None]))
    c = d[0, 0].cpu().numpy()
    c /= np.linalg.norm(c)
    rng = np.random.default_rng(94)
    away = rng.normal(size=(1024, 3))
    away /= np.linalg.norm(away, axis=1)[:, None]
    away = np.where((away @ c > 0)[:, None], -away, away) - c
    away /= np.linalg.norm(away, axis=1)[:, None]
    half = np.full(1025, 0.01)
    centre = np.concatenate([away, c[None]])
    norm = _dev_x(torch, synth.rect_normals(centre, *synth.tangent_basis(centre), half, half))
    normals = torch.empty((n_frames, 1, 4, 3), dtype=torch.float64, device="cuda")
    whole = n_frames // 1024 * 1024
    normals[:whole].view(-1, 1024, 4, 3).copy_(norm[:1024].expand(whole // 1024, 1024, 4, 3))
    normals[whole:, 0] = norm[:n_frames - whole]
    hold = [0, 77, n_frames // 2, n_frames - 2, n_frames - 1]
    normals[hold, 0] = norm[1024]
    t = torch.full((n_frames,), 1.5, dtype=torch.float64, device="cuda")
    frames = api.DeviceFrames(t, _dev_x(torch, obs).expand(n_frames, 3).contiguous(), normals)
    b = api.Batches(torch.arange(n_frames, dtype=torch.int32, device="cuda"),
                    torch.tensor([0, n_frames], dtype=torch.int32, device="cuda"), _dev_x(torch, [1.5]), np.array([1.5]))
    pf, ps, po = api.fov_check(eph, x, b, frames, pairs_cap=1000)
    assert pf.tolist() == hold and not ps.any() and not po.any()
    del normals, frames, t, b
    torch.cuda.empty_cache()


def test_fov_capacity_and_empty(torch_cuda, orc):
    torch, api = torch_cuda
    from paper_2509_04666_amd import _lib
    case = synth.tiny_case(n_obj=500, n_frames=50, n_targeted=100)
    fr = case.frames
    order, off, t_ref = orc.make_batches(fr.t)
    xe, st, _ = orc.propagate(case.ephem, case.x0, 0.0, t_ref)
    opairs = orc.fov(case.ephem, xe, st, order, off, t_ref, fr.t, fr.obs, fr.normals)
    eph = api.DeviceEphemeris.from_synth(case.ephem)
    b = api.Batches.from_host(order.astype(np.int32), off.astype(np.int32), t_ref)
    with pytest.raises(_lib.KeteError) as e:
        api.fov_check(eph, _dev_x(torch, xe), b, api.DeviceFrames.from_synth(fr), pairs_cap=3)
    assert e.value.code == _lib.KETE_ECAPACITY
    # objects far from every frame: no pairs
    far = xe.copy()
    far[..., :3] += 500.0
    pf, ps, po = api.fov_check(eph, _dev_x(torch, far), b, api.DeviceFrames.from_synth(fr))
    assert pf.numel() == 0
    # failed objects are skipped
    status = torch.zeros(500, dtype=torch.int32, device="cuda")
    status[opairs[2]] = 1
    pf, ps, po = api.fov_check(eph, _dev_x(torch, xe), b, api.DeviceFrames.from_synth(fr), status)
    assert pf.numel() == 0


def _kepler_updates(mu, x, dt, n):
    """Relative sizes [n, ...] of the first n updates of the documented
    universal-variable solve (Laguerre-Conway of order 5 from sqrt(mu) dt / r0)
    of states x [N, 6] over dt [Q, 1], in double precision, and where the
    rounding of F moves the last of them by less than the rule's 4 ulps (8 u, u
    = 2^-53): the terms of F round by some 3 u of their size while the series
    of c1..c3 are summed as they are (|z| <= 0.1), so where the sum of their
    sizes is at most 8/3 of |F' chi|."""
    smu = math.sqrt(mu)
    r0 = np.linalg.norm(x[:, :3], axis=1)
    s0 = np.sum(x[:, :3] * x[:, 3:], axis=1) / smu
    alpha = 2.0 / r0 - np.sum(x[:, 3:] ** 2, axis=1) / mu
    chi = smu * dt / r0
    out = []
    for _ in range(n):
        z = alpha * chi * chi
        sz = np.sqrt(np.abs(z)) + 1e-300
        with np.errstate(over="ignore", invalid="ignore"):
            c0 = np.where(z > 0, np.cos(sz), np.cosh(sz))
            c1 = np.where(z > 0, np.sin(sz), np.sinh(sz)) / sz
            small = np.abs(z) < 1e-3
            c2 = np.where(small, 0.5 - z / 24 + z * z / 720, (1.0 - c0) / np.where(small, 1.0, z))
            c3 = np.where(small, 1.0 / 6 - z / 120 + z * z / 5040, (1.0 - c1) / np.where(small, 1.0, z))
            terms = [r0 * chi * c1, s0 * chi ** 2 * c2, chi ** 3 * c3, -smu * dt]
            F = sum(terms)
            Fp = r0 * c0 + s0 * chi * c1 + chi ** 2 * c2
            Fpp = s0 * c0 + (1.0 - alpha * r0) * chi * c1
            exact = sum(np.abs(t) for t in terms) <= 8.0 / 3.0 * np.abs(Fp * chi)
            exact &= np.abs(z) <= 0.1
            den = Fp + np.copysign(np.sqrt(np.abs(16.0 * Fp * Fp - 20.0 * F * Fpp)), Fp)
            dx = 5.0 * F / den
            chi = chi - dx
            out.append(np.abs(dx / chi))
    return np.array(out), exact


def _one_hop_each(torch, api, cap):
    """States about a fixed Sun (ellipses up to e = 0.99 and hyperbolae, any
    place of the orbit), hop lengths from 15 minutes to 100 years, and the
    directions with kepler_iter = cap from an observer at the Sun, light being
    so fast that each direction is one hop."""
    rng = np.random.default_rng(93)
    n = 2000
    e = np.where(np.arange(n) < 1600, rng.uniform(0.0, 0.99, n), rng.uniform(1.02, 3.0, n))
    q = 0.05 * 60.0 ** rng.uniform(size=n)
    nu = np.where(e < 1, rng.uniform(-3.1, 3.1, n), rng.uniform(-1.2, 1.2, n))
    r, h = q * (1 + e) / (1 + e * np.cos(nu)), np.sqrt(synth.GM_SUN / (q * (1 + e)))
    zero = np.zeros(n)
    x = np.stack([r * np.cos(nu), r * np.sin(nu), zero, -h * np.sin(nu), h * (e + np.cos(nu)), zero], axis=1)
    dt = 10.0 ** rng.uniform(-2.0, np.log10(36500.0), 64)
    eph = api.DeviceEphemeris.from_synth(synth.sun_only_ephemeris(0.0, 4570))
    d, _ = api.lighttime_directions(eph, _dev_x(torch, x), 0.0, _dev_x(torch, dt), _dev_x(torch, np.zeros((64, 3))),
                                    api.default_opts(kepler_iter=cap, c_light=1e20))
    return x, dt[:, None], d.cpu().numpy()


@pytest.mark.parametrize("cap", [1, 2, 3, 4, 6])
def test_kepler_cap_counts_the_documented_updates(torch_cuda, cap):
    """A hop under a small cap fails exactly where the documented solve has
    not met its rule (an update within 4 ulps, or below 1e-12 and no longer
    shrinking) by that update, where rounding leaves no doubt."""
    torch, api = torch_cuda
    x, dt, d = _one_hop_each(torch, api, cap)
    failed = np.isnan(d).any(axis=2)
    u, exact = _kepler_updates(synth.GM_SUN, x, dt, cap)
    assert np.isfinite(u).all(axis=0).mean() > 0.95          # (the rest overflow)
    with np.errstate(invalid="ignore"):
        surely_fails = (u > 1e-11).all(axis=0)
        surely_ends = (u < 2e-17).any(axis=0) & exact
    _say(f"cap {cap}: {failed.sum()} of {failed.size} fail; sure {surely_fails.sum()} + {surely_ends.sum()}")
    assert failed[surely_fails].all()
    # (the terms' roundings seldom add up to more: 1 of 32,849 on the CPU)
    assert surely_ends.sum() == 0 or failed[surely_ends].mean() < 1e-3


def test_kepler_short_hops_agree_with_the_general_solve(torch_cuda):
    """The default cap, where short hops take their quicker solve, against a
    cap one lower, where every hop goes by the general one: nothing fails that
    the general solve solves, no hop of a few days fails at all, and the
    directions are the same."""
    torch, api = torch_cuda
    x, dt, d = _one_hop_each(torch, api, 60)
    _, _, g = _one_hop_each(torch, api, 59)
    bad, bad_g = np.isnan(d).any(axis=2), np.isnan(g).any(axis=2)
    short = dt * math.sqrt(synth.GM_SUN) < 0.05 * np.linalg.norm(x[:, :3], axis=1) ** 1.5
    both = ~bad & ~bad_g
    rel = np.linalg.norm(d - g, axis=2)[both] / np.linalg.norm(g, axis=2)[both]
    _say(f"default cap {bad.sum()} of {bad.size} fail, one lower {bad_g.sum()}; short {short.mean():.2f}; "
         f"max rel {rel.max():.2e}")
    assert short.mean() > 0.2 and not bad[short].any() and not bad_g[short].any()
    assert not (bad & ~bad_g).any()
    assert rel.max() < 1e-14


def test_kepler_cap_forced_from_the_host(torch_cuda, orc):
    """Host-forced non-convergence (kepler_iter = 1): every object whose
    hop the membership test needs (pairs the linear-motion bound leaves
    undecided) gets KETE_ST_KEPLER_NOCONV and loses all of its pairs, so
    what remains is a subset of the default run's pairs from unflagged
    objects only (the oracle, which hops every pair, fails everything with
    its own cap); magnitudes, light-time directions and the adjoint report
    NaN / the status; with the default cap nothing fails."""
    torch, api = torch_cuda
    from paper_2509_04666_amd import _lib
    case = synth.tiny_case(n_obj=400, n_frames=40, n_targeted=120)
    # 24 more frames, each with an edge through the oracle's apparent
    # direction of one body: no motion bound decides such a pair, so each
    # of these bodies needs a hop
    rng = np.random.default_rng(11)
    pick = rng.choice(400, 24, replace=False)
    te = rng.uniform(1.0, case.span - 1.0, 24)
    oe = synth.circular_observer(case.model, te)
    h = np.full(24, math.radians(0.75))
    nrm = np.zeros((24, 1, 4, 3))
    fr = synth.Frames.concat([case.frames, synth.Frames(te, oe, None, None, None, None, None, nrm)])
    srt = np.argsort(fr.t, kind="stable")
    fr = fr.subset(srt)
    order, off, t_ref = orc.make_batches(fr.t)
    xe, st, _ = orc.propagate(case.ephem, case.x0, 0.0, t_ref)
    pos = np.argsort(srt)[case.frames.t.size:]      # where the new frames went
    for k, f in enumerate(pos):
        b = int(np.searchsorted(off, int(np.nonzero(order == f)[0][0]), side="right") - 1)
        d = orc.lighttime(case.ephem, t_ref[b], xe[b, pick[k]], fr.t[f], fr.obs[f])[1]
        d = d / np.linalg.norm(d)
        e = synth.tangent_basis(d)[0]
        c = math.cos(h[k]) * d + math.sin(h[k]) * e
        u = math.cos(h[k]) * e - math.sin(h[k]) * d
        fr.normals[f, 0] = synth.rect_normals(c, u, np.cross(c, u), h[k], h[k])
        assert abs(fr.normals[f, 0, 1] @ d) < 1e-15
    case = dataclasses.replace(case, frames=fr)
    eph = api.DeviceEphemeris.from_synth(case.ephem)
    dfr = api.DeviceFrames.from_synth(fr)
    b = api.Batches.from_host(order.astype(np.int32), off.astype(np.int32), t_ref)
    xd = _dev_x(torch, xe)
    s0 = torch.zeros(400, dtype=torch.int32, device="cuda")
    pf, ps, po = api.fov_check(eph, xd, b, dfr, s0)
    assert pf.numel() > 50 and int(s0.abs().sum()) == 0
    o = orc.fov(case.ephem, xe, st, order, off, t_ref, fr.t, fr.obs, fr.normals, return_status=True)
    assert not o[4].any()
    _say(f"kepler cap: default run {pf.numel()} pairs (oracle {len(o[0])})")
    capped = api.default_opts(kepler_iter=1)
    s1 = torch.zeros(400, dtype=torch.int32, device="cuda")
    pf1, ps1, po1 = api.fov_check(eph, xd, b, dfr, s1, capped)
    s1h = s1.cpu().numpy()
    had = np.unique(po.cpu().numpy())
    _say(f"kepler cap 1: {pf1.numel()} pairs, {np.count_nonzero(s1h)} objects flagged, {had.size} had pairs")
    assert np.count_nonzero(s1h) > 0 and np.all(s1h[pick] != 0)
    assert set(np.unique(s1h).tolist()) <= {0, _lib.ST_KEPLER_NOCONV}
    kept = set(zip(pf1.cpu().tolist(), ps1.cpu().tolist(), po1.cpu().tolist()))
    assert kept <= set(zip(pf.cpu().tolist(), ps.cpu().tolist(), po.cpu().tolist()))
    assert all(s1h[j] == 0 for _, _, j in kept)
    # the same without a status array: the same pairs
    pf2, ps2, po2 = api.fov_check(eph, xd, b, dfr, None, capped)
    assert set(zip(pf2.cpu().tolist(), ps2.cpu().tolist(), po2.cpu().tolist())) == kept
    # magnitudes of the default run's pairs: NaN under the cap, finite without it
    H, G = synth.hg_params(np.random.default_rng(42), 400)
    Hd = torch.as_tensor(H, device="cuda")
    Gd = torch.as_tensor(G, device="cuda")
    v = api.pair_magnitudes(eph, xd, b, dfr, pf, po, Hd, Gd)
    v1 = api.pair_magnitudes(eph, xd, b, dfr, pf, po, Hd, Gd, opts=capped)
    assert torch.isfinite(v).all() and torch.isnan(v1).all()
    # light-time directions
    d, tau = api.lighttime_directions(eph, xd[0], float(t_ref[0]), torch.as_tensor(fr.t[:3], device="cuda"),
                                      torch.as_tensor(fr.obs[:3], device="cuda"), capped)
    assert torch.isnan(d).all() and torch.isnan(tau).all()
    # adjoint: every object's hops fail, so status NOCONV, NaN sky, zero gradient
    g = synth.gradient_case(n_obj=64, k_obs=5, arc=20.0)
    ctx = api.AdjointContext(api.DeviceEphemeris.from_synth(g.ephem), g.t0, g.arc,
                             torch.as_tensor(g.t_obs, device="cuda"), torch.as_tensor(g.obs_pos, device="cuda"),
                             5.0, capped)
    x0 = torch.as_tensor(g.x0, device="cuda").requires_grad_(True)
    sky = api.AdjointSky.apply(x0, ctx)
    assert torch.isnan(sky).all()
    assert np.all(ctx.status.cpu().numpy() == _lib.ST_KEPLER_NOCONV)
    sky.nan_to_num(0.0).sum().backward()
    assert torch.equal(x0.grad, torch.zeros_like(x0))


def _random_layout_frames(rng, fr, n_sub=16):
    """The frames of `fr` with their sub-frames replaced by n_sub
    rectangles of random size (0.2-1.5 deg half-sides), roll and place
    (within 4 deg of the frame centre): overlaps and gaps, no grid."""
    from paper_2509_04666_amd import synth as S
    F = fr.t.size
    # frame centre: the normalised sum of the first sub-frame's inward normals
    c = fr.normals[:, 0].sum(axis=1)
    c /= np.linalg.norm(c, axis=1, keepdims=True)
    e, n = S.tangent_basis(c)
    out = np.empty((F, n_sub, 4, 3))
    for s in range(n_sub):
        off = rng.uniform(-np.radians(4.0), np.radians(4.0), (F, 2))
        cs = c + off[:, :1] * e + off[:, 1:] * n
        cs /= np.linalg.norm(cs, axis=1, keepdims=True)
        es, ns = S.tangent_basis(cs)
        roll = rng.uniform(0, np.pi, F)[:, None]
        u = np.cos(roll) * es + np.sin(roll) * ns
        w = -np.sin(roll) * es + np.cos(roll) * ns
        hu = np.radians(rng.uniform(0.2, 1.5, F))
        hw = np.radians(rng.uniform(0.2, 1.5, F))
        out[:, s] = S.rect_normals(cs, u, w, hu, hw)
    return S.Frames(fr.t, fr.obs, None, None, None, None, None, out)


def test_fov_multi_subframe_layouts(torch_cuda, orc):
    """Frames of many sub-frames, which the sub-frame locator prunes:
    ground footprints of 8 x 8 sub-frames, and the same frames with 16 or
    120 rectangles of random size, roll and place (overlapping, with gaps;
    120 fills both mask words and gives pairs more candidate sub-frames
    than the drains list in LDS), against the oracle's brute force, given
    the oracle's states."""
    torch, api = torch_cuda
    case = synth.footprint_case(n_obj=4000, n_frames=1500, span=12.0)
    layouts = [("footprints 8x8", case.frames),
               ("random 16", _random_layout_frames(np.random.default_rng(81), case.frames)),
               ("random 120", _random_layout_frames(np.random.default_rng(82), case.frames, n_sub=120))]
    order, off, t_ref = orc.make_batches(case.frames.t)
    xe, st, _ = orc.propagate(case.ephem, case.x0, 0.0, t_ref)
    assert not st.any()
    eph = api.DeviceEphemeris.from_synth(case.ephem)
    b = api.Batches.from_host(order.astype(np.int32), off.astype(np.int32), t_ref)
    for label, fr in layouts:
        opf, ops, opo, oedge = orc.fov(case.ephem, xe, st, order, off, t_ref, fr.t, fr.obs, fr.normals)
        pf, ps, po, stats = api.fov_check(eph, _dev_x(torch, xe), b, api.DeviceFrames.from_synth(fr), None,
                                          return_stats=True)
        _say(f"{label}: stats {stats.tolist()}")
        gp = (pf.cpu().numpy(), ps.cpu().numpy(), po.cpu().numpy())
        assert np.all(np.diff(gp[0].astype(np.int64) * 2 ** 32 + gp[1].astype(np.int64) * 2 ** 25 + gp[2]) > 0)
        extra = _compare_pairs(gp, (opf, ops, opo), oedge, label)
        for p in extra:
            assert abs(_edge_of(orc, case.ephem, xe, order, off, t_ref, fr, p)) < MAS
        assert len(opf) > 500
