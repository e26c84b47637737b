"""GPU parity of the HIP solver against the FP64 oracle, through the C ABI.

Bar (FP32 kernels vs FP64 oracle): relative L2 <= 1e-4 per trace component
(p, vx, vy, vz) over all receivers and samples.  Derivative operators alone:
<= 2e-5 relative (a few FP32 FFT round-offs).
"""
import dataclasses
import math

import numpy as np
import pytest

import oracle
from paper_1705_04874_amd import inputs
from tests import physics

pytestmark = pytest.mark.gpu

TOL = 1e-4


def rel(a, b):
    return float(np.linalg.norm(np.asarray(a, np.float64) - b) / np.linalg.norm(b))


def say(*a):
    print(*a, flush=True)


@pytest.fixture(scope="module")
def B(gpu):
    from paper_1705_04874_amd import binding
    return binding


def hetero(shape, seed, water=0):
    rng = np.random.default_rng(seed)
    vp = 2400 + 900 * rng.random(shape)
    vs = vp / (1.7 + 0.3 * rng.random(shape))
    rho = 1800 + 600 * rng.random(shape)
    vp[:water], vs[:water], rho[:water] = 1500.0, 0.0, 1000.0
    return vp, vs, rho


# ---------------------------------------------------------------------------
@pytest.mark.parametrize("shape", [(24, 40, 48), (16, 75, 32), (20, 24, 60)])
def test_derivatives_match_oracle(B, shape):
    import torch
    say("derivs", shape)
    h = (10.0, 12.5, 8.0)
    vp, vs, rho = hetero(shape, 1)
    dt = 0.6e-3
    s = B.Solver(vp, vs, rho, h, dt, pml=2, kspace=1)
    s.set_sources([0, 0], np.zeros((0, 3)), np.zeros((0, 6)), np.zeros((0, 1)))
    rng = np.random.default_rng(2)
    axes_v = [(0, +1, 0), (1, -1, 3), (2, -1, 4), (0, -1, 3), (1, +1, 1), (2, -1, 5), (0, -1, 4), (1, -1, 5),
              (2, +1, 2)]
    axes_s = [(0, -1, 0), (1, -1, 1), (2, -1, 2), (1, +1, 0), (0, +1, 1), (2, +1, 0), (0, +1, 2), (2, +1, 1),
              (1, +1, 2)]
    for phase, nin, table in [(0, 6, axes_v), (1, 3, axes_s)]:
        f = rng.standard_normal((nin,) + shape)
        got = s.derivs(phase, torch.from_numpy(f.astype(np.float32)).cuda()).cpu().numpy()
        for o, (axis, sign, src) in enumerate(table):
            ref = oracle.deriv(f[src], axis, sign, h=h, kspace=1, c_ref=vp.max(), dt=dt)
            e = rel(got[o], ref)
            assert e < 2e-5, (phase, o, e)


# ---------------------------------------------------------------------------
def run_both(B, w, nt, **over):
    s = B.Solver.from_workload(w, **over)
    s.set_workload_sources(w)
    g = s.run(nt).cpu().numpy()
    refs = [oracle.run_shot(w, shot=k, nt=nt, **over) for k in range(w.n_shots)]
    s.close()
    return g, refs


def test_two_layer_32_full(B):
    w = inputs.two_layer_workload()
    say("two layer", w.model.shape, w.nt)
    g, refs = run_both(B, w, w.nt)
    for c in range(4):
        e = rel(g[0, c], refs[0][c])
        say(f"  comp {c} rel-L2 {e:.3e}")
        assert e <= TOL


def small_workload(shape=(30, 24, 40), nt=150, kspace=1, shots=2, seed=3, pml=6):
    nz, ny, nx = shape
    vp, vs, rho = hetero(shape, seed, water=5)
    m = inputs.Model(vp, vs, rho)
    dt = 0.8e-3
    rec = np.concatenate([inputs.receiver_block(4, nx - 4, 3, ny - 3, 5),
                          np.array([[nx - 1, ny - 1, nz - 1], [0, 0, 0]], np.int32)])
    rng = np.random.default_rng(seed)
    ijk, mts, ofs = [], [], [0]
    for k in range(shots):
        for q in range(k + 1):
            ijk.append([rng.integers(8, nx - 8), rng.integers(6, ny - 6), rng.integers(10, nz - 8)])
            mts.append(inputs.random_dc(rng, 1000.0) + (q == 1) * inputs.clvd(300.0))
        ofs.append(len(ijk))
    # one source at a grid corner: shear stencil wraps around the periodic edges
    ijk.append([0, 0, nz - 1])
    mts.append(inputs.double_couple(0.5, 0.9, 0.2, 800.0))
    ofs[-1] = len(ijk)
    wav = np.stack([inputs.ricker(30.0 + 3 * q, dt, nt) for q in range(len(ijk))])
    return inputs.Workload("small", m, (10.0, 10.0, 10.0), dt, nt, pml, 2.0, kspace, 0.0, rec,
                           np.array(ijk, np.int32), np.array(mts), np.array(ofs, np.int32), wav)


@pytest.mark.parametrize("kspace", [1, 0])
def test_small_heterogeneous_multishot(B, kspace):
    w = small_workload(kspace=kspace)
    say("small multishot kspace", kspace, w.model.shape, w.n_shots)
    g, refs = run_both(B, w, w.nt)
    for k in range(w.n_shots):
        for c in range(4):
            e = rel(g[k, c], refs[k][c])
            say(f"  shot {k} comp {c} rel-L2 {e:.3e}")
            assert e <= TOL


def test_shots_are_independent(B):
    """Batched shots give exactly the traces of the same shots run one at a time."""
    w = small_workload(nt=60, shots=3)
    s = B.Solver.from_workload(w)
    s.set_workload_sources(w)
    batch = s.run(w.nt).cpu().numpy()
    for k in range(w.n_shots):
        a, b = int(w.shot_ofs[k]), int(w.shot_ofs[k + 1])
        s1 = B.Solver.from_workload(w)
        s1.set_tuning(**s.tuning_values())   # the same launch shapes: identical arithmetic
        s1.set_sources([0, b - a], w.src_ijk[a:b], w.src_m[a:b], w.wavelet[a:b])
        one = s1.run(w.nt).cpu().numpy()[0]
        np.testing.assert_array_equal(batch[k], one)


def test_run_is_stateful_and_checkpoint_is_exact(B):
    w = small_workload(nt=80, shots=1)
    s = B.Solver.from_workload(w)
    s.set_workload_sources(w)
    full = s.run(80).cpu().numpy()
    s.set_workload_sources(w)
    a = s.run(30).cpu().numpy()
    st = s.get_state()
    b = s.run(50).cpu().numpy()
    np.testing.assert_array_equal(np.concatenate([a, b], axis=3), full)
    s2 = B.Solver.from_workload(w)
    s2.set_tuning(**s.tuning_values())
    s2.set_workload_sources(w)
    s2.set_state(st, 30)
    c = s2.run(50).cpu().numpy()
    np.testing.assert_array_equal(c, b)


def test_undamped_cells_hold_each_field_in_its_first_part(B):
    """The cells the absorbing layer leaves undamped (every factor of the split
    update exactly 1) are those with every index in [pml, n - 2 - pml] (at
    pml - 1 and n - 1 - pml a half node is damped), all cells without a layer.
    After a run they hold each field in its first split part, the other parts
    exactly zero; set_state sums a given state's parts there and leaves the
    damped cells as given."""
    w = small_workload(nt=60, shots=1)
    nz, ny, nx = w.model.shape
    L = w.pml
    s = B.Solver.from_workload(w)
    lo, hi = s.undamped_range()
    assert lo == (L, L, L) and hi == (nx - 2 - L, ny - 2 - L, nz - 2 - L), (lo, hi)
    mask = physics.undamped_mask(w.model.shape, lo, hi)
    s.set_workload_sources(w)
    s.run(w.nt)
    st = s.get_state()
    for _, f0, n in physics.FIELD_PARTS:
        assert np.abs(st[f0][mask]).max() > 0
        for k in range(1, n):
            assert not st[f0 + k][mask].any()
    given = np.random.default_rng(5).standard_normal(st.shape).astype(np.float32)
    s.set_state(given, 0)
    back = s.get_state()
    np.testing.assert_allclose(back, physics.collapse_undamped(given, mask), rtol=0, atol=1e-6)
    np.testing.assert_array_equal(back[:, ~mask], given[:, ~mask])
    s.close()
    n0 = B.Solver(w.model.vp, w.model.vs, w.model.rho, w.d, w.dt, pml=0)
    assert n0.undamped_range() == ((0, 0, 0), (nx - 1, ny - 1, nz - 1))
    n0.close()


@pytest.mark.parametrize("wave", ["P", "S"])
def test_plane_wave(B, wave):
    shape = (24, 20, 32)
    h = (10.0, 12.5, 8.0)
    vp, vs, rho, dt = 3000.0, 1700.0, 2300.0, 0.4e-3
    s = B.Solver(np.full(shape, vp), np.full(shape, vs), np.full(shape, rho), h, dt, pml=0, kspace=1, c_ref=vp)
    s.set_sources([0, 0], np.zeros((0, 3)), np.zeros((0, 6)), np.zeros((0, 1)))
    s.set_state(physics.plane_wave_state(shape, h, dt, (3, 2, 1), wave, vp, vs, rho, 0, 1, vp), 0)
    s.run(200)
    got = physics.summed(s.get_state().astype(np.float64))
    want = physics.summed(physics.plane_wave_state(shape, h, dt, (3, 2, 1), wave, vp, vs, rho, 200, 1, vp))
    vscale = max(np.abs(b).max() for b in want[:3])
    sscale = max(np.abs(b).max() for b in want[3:])
    for i, (a, b) in enumerate(zip(got, want)):
        scale = vscale if i < 3 else sscale
        assert np.abs(a - b).max() < 2e-4 * scale, (i, np.abs(a - b).max() / scale)


def test_error_codes(B):
    shape = (16, 16, 16)
    vp, vs, rho = [np.full(shape, v) for v in (3000.0, 1700.0, 2300.0)]
    limit = 2 / math.pi * 10.0 / (3000.0 * math.sqrt(3))
    with pytest.raises(B.PstdError) as e:
        B.Solver(vp, vs, rho, (10, 10, 10), 1.05 * limit, kspace=0, pml=2)
    assert e.value.code == B.PSTD_EUNSTABLE
    shp = (16, 16, 17)
    with pytest.raises(B.PstdError) as e:
        B.Solver(np.full(shp, 3000.0), np.full(shp, 1700.0), np.full(shp, 2300.0), (10, 10, 10), 1e-3, pml=2)
    assert e.value.code == B.PSTD_EUNSUPPORTED
    s = B.Solver(vp, vs, rho, (10, 10, 10), 1e-3, pml=2)
    with pytest.raises(B.PstdError) as e:
        s.set_sources([0, 1], np.array([[0, 0, 16]]), np.zeros((1, 6)), np.zeros((1, 4)))
    assert e.value.code == B.PSTD_EINVAL


def test_graph_replay_equals_eager(B, monkeypatch):
    w = small_workload(nt=41, shots=2)
    s = B.Solver.from_workload(w)
    s.set_workload_sources(w)
    monkeypatch.setenv("PSTD_GRAPH", "1")
    g = s.run(41).cpu().numpy()
    s.reset()
    monkeypatch.setenv("PSTD_GRAPH", "0")
    e = s.run(41).cpu().numpy()
    np.testing.assert_array_equal(g, e)
    # a second call continues from step 41 in both modes
    monkeypatch.setenv("PSTD_GRAPH", "1")
    g2 = s.run(10).cpu().numpy()
    s.reset()
    monkeypatch.setenv("PSTD_GRAPH", "0")
    s.run(41)
    e2 = s.run(10).cpu().numpy()
    np.testing.assert_array_equal(g2, e2)


def test_run_many_uneven_grids(B):
    """Several models of different sizes advanced together equal separate runs."""
    ws = [small_workload(shape=(30, 24, 40), nt=50, shots=1, seed=4),
          small_workload(shape=(24, 32, 48), nt=50, shots=2, seed=5),
          small_workload(shape=(40, 30, 32), nt=50, shots=1, seed=6)]
    solos, tunings = [], []
    for w in ws:
        s = B.Solver.from_workload(w)
        s.set_workload_sources(w)
        solos.append(s.run(50).cpu().numpy())
        tunings.append(s.tuning_values())
    ss = []
    for w, tu in zip(ws, tunings):
        s = B.Solver.from_workload(w)
        s.set_tuning(**tu)
        s.set_workload_sources(w)
        ss.append(s)
    outs = B.run_many(ss, 50)
    for a, b in zip(outs, solos):
        np.testing.assert_array_equal(a.cpu().numpy(), b)


def test_every_tuning_value_gives_the_same_traces(B):
    """The autotuner may pick any built launch shape: y / z tile widths and the
    update kernels' threads per block.  Each computes every pencil with the
    same butterflies and every cell with the same update, so the traces agree
    to FP32 rounding (fused multiply-adds may be contracted differently)."""
    w = small_workload(shape=(48, 128, 64), nt=30, shots=2, seed=8)
    s = B.Solver.from_workload(w)
    s.set_workload_sources(w)
    t = s.tuning()
    say("tuning", t)
    for k in B.TUNE_KNOBS:
        cand = t[k + "_candidates"]
        assert t[k] in cand
        # the chosen value was measured and is the fastest measured
        assert cand[t[k]] == min(v for v in cand.values() if v > 0), k
    assert len(t["y_tile_candidates"]) >= 2 and len(t["z_tile_candidates"]) >= 2
    assert len(t["vel_threads_candidates"]) >= 2
    ref = s.run(w.nt).cpu().numpy()
    scale = np.abs(ref).max(axis=(2, 3), keepdims=True)
    combos = [dict(y_tile=y, z_tile=z, vel_threads=256, str_threads=256)
              for y in t["y_tile_candidates"] for z in t["z_tile_candidates"]]
    combos += [dict(y_tile=16, z_tile=16, vel_threads=v, str_threads=v) for v in t["vel_threads_candidates"]]
    # the z kernels' thread counts with every tile they are built for, and both field groupings
    for z in t["z_tile_candidates"]:
        for zt in t["z_threads_candidates"]:
            for zf in t["z_fields_candidates"]:
                combos.append(dict(y_tile=16, z_tile=z, vel_threads=256, str_threads=256, z_threads=zt, z_fields=zf))
    for kw in combos:
        try:
            s.set_tuning(**kw)
        except B.PstdError as e:
            # a z thread count that is not built for that tile
            assert e.code == B.PSTD_EUNSUPPORTED and kw.get("z_threads", 256) != 256, kw
            continue
        got_t = s.tuning()
        assert all(got_t[k] == v for k, v in kw.items())
        s.reset()
        got = s.run(w.nt).cpu().numpy()
        err = np.abs(got - ref).max(axis=(2, 3), keepdims=True) / scale
        assert err.max() < 1e-5, (kw, float(err.max()))
    with pytest.raises(B.PstdError) as e:
        s.set_tuning(y_tile=7)
    assert e.value.code == B.PSTD_EUNSUPPORTED


@pytest.mark.parametrize("shape", [(20, 16, 75), (24, 20, 125)])
def test_odd_x_lengths_against_oracle(B, shape):
    """Odd x lengths (no Nyquist plane in the x half spectrum), odd y, and
    anisotropic spacing: traces against the FP64 oracle."""
    w = small_workload(shape=shape, nt=60, shots=1, seed=9, pml=4)
    w.d = (12.5, 11.0, 9.0)
    say("odd x", shape)
    g, refs = run_both(B, w, w.nt)
    for c in range(4):
        e = rel(g[0, c], refs[0][c])
        say(f"  comp {c} rel-L2 {e:.3e}")
        assert e <= TOL


def test_paper_shaped_grid_initial_pressure_source(B):
    """The paper's 125 x 75 x 300 grid with 12.5 / 12.5 / 10 m cells and an
    initial-pressure source of 1 Pa smoothed by the Blackman window in k-space:
    the pressure at the source cell after the first step is the window's centre
    weight 0.42^3 Pa, and 40 steps agree with the FP64 oracle (which smooths
    with its own FFT) at receivers around the source."""
    w = inputs.paper_shaped_workload(nt=40)
    sx, sy, sz = w.src_ijk[0]
    near = np.array([[sx + dx, sy + dy, sz + dz] for dx in (-3, 0, 3) for dy in (-2, 0, 2) for dz in (-4, 0, 4)],
                    np.int32)
    s = B.Solver.from_workload(w, rec=near)
    s.set_workload_sources(w)
    g = s.run(w.nt).cpu().numpy()[0]
    s.close()
    ref = oracle.run_shot(w, nt=w.nt, rec=near)
    centre = 13                                              # (dx, dy, dz) = (0, 0, 0)
    assert abs(ref[0][centre, 0] - 0.42 ** 3) < 1e-12       # p right after the smoothed 1 Pa initial stress
    assert abs(g[0][centre, 0] - 0.42 ** 3) < 1e-6
    for c in range(4):
        e = rel(g[c], ref[c])
        say(f"  paper-shaped comp {c} rel-L2 {e:.3e}")
        assert e <= TOL


def test_blackman_smoothed_sources_against_oracle(B):
    """Sources smoothed by the Blackman window in k-space (the GPU injects the
    equivalent 5-point stencil per axis, the oracle multiplies the delta's
    spectrum with its own FFT), including a source next to a grid corner whose
    stencil wraps around the periodic edges."""
    w = small_workload(nt=80, shots=2, seed=14)
    w.smooth = 1
    say("smoothed sources", w.model.shape, w.n_shots)
    g, refs = run_both(B, w, w.nt)
    for k in range(w.n_shots):
        for c in range(4):
            e = rel(g[k, c], refs[k][c])
            say(f"  shot {k} comp {c} rel-L2 {e:.3e}")
            assert e <= TOL


@pytest.mark.parametrize("shape,smooth", [((30, 24, 20), 1), ((30, 75, 75), 1), ((20, 24, 128), 1), ((30, 75, 75), 0)])
def test_injected_stress_of_many_sources(B, shape, smooth):
    """Source injection where a wave's rows hold more entries than it has lanes
    and several sources add to one cell: coinciding and neighbouring sources in
    the second shot, one in the last row (whose stencil wraps), rows shorter
    than a wave, of a length that leaves a ragged last block, and longer.  From
    rest, one step leaves exactly the injected stress: up to 16 roundings of
    2^-24 per value against the oracle's state."""
    nz, ny, nx = shape
    w = small_workload(shape=shape, nt=1, shots=2, seed=17)
    w.smooth = smooth
    c = [nx // 2, ny // 2, nz - 12]
    w.src_ijk = np.array([c, c, [c[0] + 1, c[1], c[2]], [nx - 1, ny - 1, nz - 1]], np.int32)
    w.wavelet = np.random.default_rng(18).standard_normal((4, 1))
    s = B.Solver.from_workload(w)
    s.set_workload_sources(w)
    s.run(1)
    for k in range(w.n_shots):
        q = slice(w.shot_ofs[k], w.shot_ofs[k + 1])
        o = oracle.Solver.from_workload(w)
        o.set_sources(w.src_ijk[q], w.src_m[q], w.wavelet[q])
        o.run(1)
        got, ref = physics.summed(s.get_state(k).astype(np.float64)), physics.summed(o.get_state())
        for f in range(3, 9):
            e = rel(got[f], ref[f])
            say(f"  {shape} smooth {smooth} shot {k} stress {f - 3} rel-L2 {e:.3e}")
            assert e <= 16 * 2.0 ** -24
        o.close()
    s.close()


# ---------------------------------------------------------------------------
def viscous_workload(nt=150, shots=2, seed=21, kspace=1):
    """The small heterogeneous workload with Kelvin-Voigt viscosities: chi and
    eta random per cell, eta = 0 in the water layer (the harmonic mean then
    gives zero shear viscosity on the nodes touching it).  chi + 2 eta stays
    near 1e6 Pa s, where dt k_max^2 (chi + 2 eta) / rho ~ 0.2: stable, and at
    the wavelet's frequencies the amplitude loss over the run is ~10 %."""
    w = small_workload(nt=nt, shots=shots, seed=seed, kspace=kspace)
    rng = np.random.default_rng(seed + 100)
    shape = w.model.shape
    w.chi = 2.0e5 + 3.0e5 * rng.random(shape)
    w.eta = 1.5e5 + 2.5e5 * rng.random(shape)
    w.eta[:5] = 0.0
    return w


@pytest.mark.parametrize("kspace", [1, 0])
def test_kelvin_voigt_viscosity_against_oracle(B, kspace):
    """Viscous stress update (eq. 1-2, backward difference of the velocity
    derivatives) against the FP64 oracle, and the loss it causes is far above
    the tolerance (the viscous terms are exercised)."""
    w = viscous_workload(kspace=kspace)
    say("viscous kspace", kspace, w.model.shape, w.n_shots)
    g, refs = run_both(B, w, w.nt)
    loss = dataclasses.replace(w, chi=None, eta=None)
    lossless = B.Solver.from_workload(loss)
    lossless.set_workload_sources(loss)
    g0 = lossless.run(w.nt).cpu().numpy()
    lossless.close()
    for k in range(w.n_shots):
        for c in range(4):
            e = rel(g[k, c], refs[k][c])
            d = rel(g0[k, c], refs[k][c])
            say(f"  shot {k} comp {c} rel-L2 {e:.3e} (lossless differs by {d:.3e})")
            assert e <= TOL
            assert d > 100 * TOL
        assert np.linalg.norm(g[k]) < np.linalg.norm(g0[k])


def test_kelvin_voigt_state_matches_oracle_and_checkpoints(B):
    """The 33 state fields (24 split parts + the previous step's nine velocity
    derivatives in the documented order) agree with the oracle's after 40
    steps, and a restored checkpoint continues bit-exactly."""
    w = viscous_workload(nt=90, shots=1)
    s = B.Solver.from_workload(w)
    assert s.n_state == 33
    s.set_workload_sources(w)
    a = s.run(40).cpu().numpy()
    st = s.get_state()
    b = s.run(50).cpu().numpy()
    o = oracle.Solver.from_workload(w)
    assert o.n_state == 33
    o.set_sources(w.src_ijk, w.src_m, w.wavelet)
    o.run(40)
    ref = o.get_state()
    o.close()
    # the undamped cells keep each field in its first split part
    ref = physics.collapse_undamped(ref, physics.undamped_mask(ref.shape[1:], *s.undamped_range()))
    for name, ef, ep in physics.split_errors(st, ref):
        assert ef <= TOL and ep <= TOL, (name, ef, ep)
    for f in range(24, 33):
        e = rel(st[f], ref[f])
        assert e <= TOL, (f, e)
    s2 = B.Solver.from_workload(w)
    s2.set_tuning(**s.tuning_values())
    s2.set_workload_sources(w)
    s2.set_state(st, 40)
    np.testing.assert_array_equal(s2.run(50).cpu().numpy(), b)
    # back to lossless: 24 state fields
    s2.set_viscosity(None, None)
    assert s2.n_state == 24
    s.close()
    s2.close()
    assert a.shape == (1, 4, w.rec.shape[0], 40)


def test_degenerate_inputs(B):
    """Empty and degenerate inputs: a shot without sources records exact zeros
    next to a live shot; a zero moment tensor records exact zeros; a wavelet
    shorter than the run equals the same wavelet zero-padded; nt = 0 is a
    no-op; a model without receivers runs; chi = eta = 0 reproduces the
    lossless traces (up to the order of two roundings)."""
    import torch
    w = small_workload(nt=40, shots=1, seed=9)
    src, m6 = w.src_ijk[:1], w.src_m[:1]
    wav = w.wavelet[:1, :40]
    s = B.Solver.from_workload(w)
    s.set_sources([0, 0, 1], src, m6, wav)
    two = s.run(40).cpu().numpy()
    assert not two[0].any() and two[1].any()
    s.set_sources([0, 1], src, np.zeros((1, 6)), wav)
    assert not s.run(40).cpu().numpy().any()
    s.set_sources([0, 1], src, m6, wav)
    full = s.run(40).cpu().numpy()
    np.testing.assert_array_equal(full[0], two[1])
    short = wav[:, :12]
    s.set_sources([0, 1], src, m6, short)
    a = s.run(40).cpu().numpy()
    padded = np.concatenate([short, np.zeros((1, 28))], axis=1)
    s.set_sources([0, 1], src, m6, padded)
    np.testing.assert_array_equal(a, s.run(40).cpu().numpy())
    step = s.step
    e = s.run(0)
    assert e.numel() == 0 and s.step == step
    n = B.Solver(w.model.vp, w.model.vs, w.model.rho, w.d, w.dt, pml=w.pml, rec=np.zeros((0, 3), np.int32))
    n.set_sources([0, 1], src, m6, wav)
    assert n.run(10).shape == (1, 4, 0, 10)
    st = n.get_state()
    assert np.isfinite(st).all() and st.any()
    z = B.Solver.from_workload(w)
    z.set_tuning(**s.tuning_values())
    z.set_viscosity(np.zeros(w.model.shape), np.zeros(w.model.shape))
    z.set_sources([0, 1], src, m6, wav)
    zv = z.run(40).cpu().numpy()
    assert float(np.abs(zv - full).max()) <= 1e-5 * float(np.abs(full).max())
    for x in (s, n, z):
        x.close()


@pytest.mark.parametrize("dt", [0.8e-3, 2.2e-3])
def test_kappa_series_against_oracle(B, monkeypatch, dt):
    """The z operator can evaluate the k-space correction as the power series of
    sin(a)/a in s = a^2 (a = c_ref |k| dt / 2) instead of reading the table.
    Both ways against the FP64 oracle; dt = 2.2 ms puts s near 4, the largest
    value the series is offered for (the corner wavenumbers), and is stable
    because the corrected scheme with c_ref >= c_max has no CFL limit."""
    w = small_workload(nt=60, shots=1, seed=12)
    w.dt = dt
    ref = oracle.run_shot(w, nt=w.nt)
    out = {}
    for mode in ("table", "series", "default"):
        if mode == "default":
            monkeypatch.delenv("PSTD_KAPPA", raising=False)   # series in the stress phase only
        else:
            monkeypatch.setenv("PSTD_KAPPA", mode)
        s = B.Solver.from_workload(w)
        s.set_workload_sources(w)
        out[mode] = s.run(w.nt).cpu().numpy()[0]
        s.close()
    for c in range(4):
        for mode in ("table", "series", "default"):
            e = rel(out[mode][c], ref[c])
            say(f"  dt {dt} {mode} comp {c} rel-L2 {e:.3e}")
            assert e <= TOL
        assert rel(out["series"][c], out["table"][c]) <= 2e-5
        assert rel(out["default"][c], out["table"][c]) <= 2e-5


def test_caller_workspace(B):
    """Shot state in caller-provided device memory: the same traces bit for bit
    (the workspace starts as garbage: set_sources clears it), the context's own
    memory shrinks by the state, a short or misaligned workspace is rejected,
    and NULL returns to the context's own memory."""
    import torch
    w = small_workload(nt=60, shots=2, seed=15)
    a = B.Solver.from_workload(w)
    a.set_workload_sources(w)
    ref = a.run(60).cpu().numpy()
    own = a.device_bytes
    b = B.Solver.from_workload(w)
    b.set_tuning(**a.tuning_values())
    need = b.workspace_size(2)
    assert need >= 2 * 24 * int(np.prod(w.model.shape)) * 4
    b.set_workspace(torch.empty(need - 256, dtype=torch.uint8, device="cuda"))
    with pytest.raises(B.PstdError) as e:
        b.set_workload_sources(w)
    assert e.value.code == B.PSTD_EINVAL
    buf = torch.full((need + 512,), 0x7f, dtype=torch.uint8, device="cuda")
    with pytest.raises(B.PstdError) as e:
        b.set_workspace(buf[1:])
    assert e.value.code == B.PSTD_EINVAL
    b.set_workspace(buf)
    b.set_workload_sources(w)
    assert b.device_bytes < own
    np.testing.assert_array_equal(b.run(60).cpu().numpy(), ref)
    b.set_workspace(None)
    b.set_workload_sources(w)
    assert b.device_bytes == own
    np.testing.assert_array_equal(b.run(60).cpu().numpy(), ref)
    a.close()
    b.close()


@pytest.mark.parametrize("nx,counts", [(16, (128, 256)), (20, (128, 256)), (24, (128, 256)), (30, (128, 256)),
                                       (32, (128, 256, 512)), (40, (128, 256)), (48, (128, 256))])
def test_update_thread_counts_of_short_rows(B, nx, counts):
    """Lengths up to 48 take update kernels of more threads than a block of
    their rows has cells (128 to 256 cells): every count can be forced, and
    three steps from a random state, with a smoothed source whose stencil wraps
    around the grid's last row and a ragged last block (1200 rows by 8, 2250 by
    8 and 4), agree with the FP64 oracle to this file's bar and with 128
    threads to FP32 rounding (as every launch shape: 1e-5 of a field's largest
    value)."""
    shape = (30, 75, nx) if nx != 20 else (16, 75, nx)
    nz, ny, _ = shape
    rng = np.random.default_rng(60 + nx)
    vp, vs, rho = hetero(shape, 61)
    src = np.array([[nx - 1, ny - 1, nz - 1], [nx // 2, 30, 9]], np.int32)
    rec = inputs.receiver_block(1, nx - 1, 3, ny - 3, 5)
    w = inputs.Workload("short_rows", inputs.Model(vp, vs, rho), (10.0, 10.0, 10.0), 0.8e-3, 3, 4, 2.0, 1, 0.0, rec,
                        src, np.stack([inputs.random_dc(rng, 1e6), inputs.random_dc(rng, 1e6)]),
                        np.array([0, 2], np.int32), rng.standard_normal((2, 3)))
    w.smooth = 1
    amp = np.where(np.arange(24) < 9, 2e-7, 1.0)[:, None, None, None]
    start = (amp * rng.standard_normal((24,) + shape)).astype(np.float32)
    s = B.Solver.from_workload(w)
    s.set_workload_sources(w)
    s.set_state(start, 0)
    start = s.get_state()   # the undamped cells' parts collapsed
    o = oracle.Solver.from_workload(w)
    o.set_sources(w.src_ijk, w.src_m, w.wavelet)
    o.set_state(start.astype(np.float64))
    o.step = 0
    o.run(3)
    ref = physics.collapse_undamped(o.get_state(), physics.undamped_mask(shape, *s.undamped_range()))
    o.close()
    got = {}
    for nt in counts:
        s.set_tuning(vel_threads=nt, str_threads=nt)
        s.set_workload_sources(w)
        t = s.tuning()
        assert t["vel_threads"] == nt and t["str_threads"] == nt
        s.set_state(start, 0)
        say("short rows", nx, nt)
        s.run(3)
        got[nt] = s.get_state()
        for name, ef, ep in physics.split_errors(got[nt], ref):
            assert ef <= TOL and ep <= TOL, (nt, name, ef, ep)
        scale = np.abs(got[128]).max(axis=(1, 2, 3))
        assert (np.abs(got[nt] - got[128]).max(axis=(1, 2, 3)) <= 1e-5 * scale).all(), nt
    s.close()


@pytest.mark.parametrize("shape", [(30, 24, 40), (20, 24, 75)])
def test_viscous_update_that_streams(B, shape):
    """Where the contexts that run together hold more than the last-level cache
    (256 MB) their update kernels pass it by.  A small viscous model beside a
    128^3 one takes that form of the viscous stress update: traces and all 33
    state fields against the oracle (this file's bar) and against the model
    alone, with every thread count of the update kernels, to FP32 rounding
    (1e-5 of a field's largest value, as for every launch shape)."""
    nt = 60
    w = small_workload(shape=shape, nt=nt, shots=1, seed=22)
    rng = np.random.default_rng(122)
    w.chi = 2.0e5 + 3.0e5 * rng.random(shape)
    w.eta = 1.5e5 + 2.5e5 * rng.random(shape)
    w.eta[:5] = 0.0
    o = oracle.Solver.from_workload(w)
    o.set_sources(w.src_ijk, w.src_m, w.wavelet)
    otr = o.run(nt)
    ref = o.get_state()
    o.close()
    big_w = inputs.layered128_shots(1, nt=nt)
    big = B.Solver.from_workload(big_w)
    big.set_workload_sources(big_w)
    assert big.workspace_size(1) > 256 << 20
    s = B.Solver.from_workload(w)
    s.set_workload_sources(w)
    assert s.n_state == 33 and s.workspace_size(1) < 128 << 20
    ref = physics.collapse_undamped(ref, physics.undamped_mask(shape, *s.undamped_range()))
    base = s.tuning_values()
    for n in s.tuning()["str_threads_candidates"]:
        s.set_tuning(**dict(base, vel_threads=n, str_threads=n))
        s.reset()
        alone, st0 = s.run(nt).cpu().numpy(), s.get_state()
        s.reset()
        big.reset()
        say("viscous beside a large model", shape, n)
        traces = B.run_many([s, big], nt)[0].cpu().numpy()
        st = s.get_state()
        for c in range(4):
            assert rel(traces[0, c], otr[c]) <= TOL, (n, c)
        for name, ef, ep in physics.split_errors(st, ref):
            assert ef <= TOL and ep <= TOL, (n, name, ef, ep)
        for f in range(24, 33):
            assert rel(st[f], ref[f]) <= TOL, (n, f)
        for a, b in ((traces[0], alone[0]), (st, st0)):
            ax = tuple(range(1, a.ndim))
            assert (np.abs(a - b).max(axis=ax) <= 1e-5 * np.abs(b).max(axis=ax)).all(), n
    s.close()
    big.close()
