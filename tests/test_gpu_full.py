"""GPU checks at the full workload sizes, in the launch configuration the bench
times (one context, graph replay of step pairs).

 * 128^3 layered model, 2000 steps, one DC source: traces at a fixed sample
   of 32 receivers against the stored FP64 oracle run (rel-L2 <= 1e-4 per
   component).
 * 384 x 384 x 256 model: the oracle cannot run it in a test, so the test uses
   properties that hold at any size: doubling the moment tensor doubles every
   trace exactly (scaling by 2 is exact in binary floating point), delaying
   the wavelet by m samples delays every trace by m samples exactly (the
   state stays exactly zero until the source starts), and the derivative
   operators at lengths 384 and 256 match the oracle on a thin grid.
   At full size the oracle can still take one step: from the GPU's state
   after 600 steps (waves in the PML on every face) one GPU step and one FP64
   oracle step agree on every cell of all 24 split fields.
 * 64 shots batched on the 128^3 model: selected shots equal the same shots
   run alone, bit for bit.
"""
import os

import numpy as np
import pytest

import oracle
from paper_1705_04874_amd import inputs
from tests import physics

pytestmark = pytest.mark.gpu

# the nine fields of the state and the indices of their split parts (the
# order of oracle.STATE_NAMES)
SPLIT_PARTS = [("vx", [0, 1, 2]), ("vy", [3, 4, 5]), ("vz", [6, 7, 8]), ("sxx", [9, 10, 11]),
               ("syy", [12, 13, 14]), ("szz", [15, 16, 17]), ("sxy", [18, 19]), ("sxz", [20, 21]),
               ("syz", [22, 23])]

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
GOLD = os.path.join(ROOT, "tests", "golden", "layered128_oracle_traces.npz")


def say(*a):
    print(*a, flush=True)


@pytest.fixture(scope="module")
def B(gpu):
    from paper_1705_04874_amd import binding
    return binding


def test_layered128_full_against_oracle_golden(B):
    if not os.path.exists(GOLD):
        pytest.fail("tests/golden/layered128_oracle_traces.npz missing (tests/golden/make_layered128_golden.py writes it)")
    g = np.load(GOLD, allow_pickle=False)
    nt = int(g["nt"])
    w = inputs.layered128_workload(nt=nt)
    from tests.golden.make_layered128_golden import model_digest
    assert str(g["digest"]) == model_digest(w), "workload generator changed since the golden was written"
    say("layered128 full", w.model.shape, nt)
    s = B.Solver.from_workload(w)
    s.set_workload_sources(w)
    tr = s.run(nt).cpu().numpy()[0][:, g["receivers"]].astype(np.float64)
    ref = g["traces"]
    for c, name in enumerate(["p", "vx", "vy", "vz"]):
        e = np.linalg.norm(tr[c] - ref[c]) / np.linalg.norm(ref[c])
        say(f"  {name}: rel-L2 {e:.3e}")
        assert e <= 1e-4


# the full-size lengths, and the largest built length (512) on each axis
@pytest.mark.parametrize("shape", [(256, 16, 384), (16, 384, 40), (16, 20, 512), (512, 16, 24), (20, 512, 16),
                                   # the lengths of the uneven-model batch (radix-5 and radix-3 plans)
                                   (16, 20, 80), (20, 144, 16), (160, 20, 16), (96, 16, 120), (16, 96, 160),
                                   (80, 120, 16), (144, 16, 20)])
def test_derivatives_at_large_lengths(B, shape):
    import torch
    say("derivs", shape)
    h = (10.0, 10.0, 10.0)
    rng = np.random.default_rng(7)
    vp = 2500 + 500 * rng.random(shape)
    vs = vp / 1.8
    rho = 310 * vp ** 0.25
    dt = 0.8e-3
    s = B.Solver(vp, vs, rho, h, dt, pml=4, kspace=1)
    s.set_sources([0, 0], np.zeros((0, 3)), np.zeros((0, 6)), np.zeros((0, 1)))
    f = rng.standard_normal((3,) + shape)
    got = s.derivs(1, torch.from_numpy(f.astype(np.float32)).cuda()).cpu().numpy()
    table = [(0, -1, 0), (1, -1, 1), (2, -1, 2), (1, +1, 0), (0, +1, 1), (2, +1, 0), (0, +1, 2), (2, +1, 1),
             (1, +1, 2)]
    for o, (axis, sign, src) in enumerate(table):
        ref = oracle.deriv(f[src], axis, sign, h=h, kspace=1, c_ref=vp.max(), dt=dt)
        e = np.linalg.norm(got[o] - ref) / np.linalg.norm(ref)
        assert e < 2e-5, (o, e)


@pytest.mark.parametrize("ny", [16, 75, 144, 240, 384])
def test_derivatives_for_every_y_tile(B, ny):
    """Both phases' nine derivatives with every built y tile forced (the inverse
    y kernel forms the x and y derivatives of one spectrum in turn, the second
    in place; 512 threads where the tile is large; at 240 the widest tile leaves
    no room for the symbol in LDS), with and without a Nyquist plane, against
    the oracle (FP32 transforms: 2e-5)."""
    import torch
    h, dt = (10.0, 12.0, 9.0), 0.8e-3
    rng = np.random.default_rng(8)
    tables = [[(0, +1, 0), (1, -1, 3), (2, -1, 4), (0, -1, 3), (1, +1, 1), (2, -1, 5), (0, -1, 4), (1, -1, 5),
               (2, +1, 2)],
              [(0, -1, 0), (1, -1, 1), (2, -1, 2), (1, +1, 0), (0, +1, 1), (2, +1, 0), (0, +1, 2), (2, +1, 1),
               (1, +1, 2)]]
    for nx in (20, 75):
        shape = (16, ny, nx)
        vp = 2500 + 500 * rng.random(shape)
        s = B.Solver(vp, vp / 1.8, 310 * vp ** 0.25, h, dt, pml=4, kspace=1)
        s.set_sources([0, 0], np.zeros((0, 3)), np.zeros((0, 6)), np.zeros((0, 1)))
        f = rng.standard_normal((6,) + shape)
        refs = [[oracle.deriv(f[src], axis, sign, h=h, kspace=1, c_ref=vp.max(), dt=dt) for axis, sign, src in t]
                for t in tables]
        for tile in s.tuning()["y_tile_candidates"]:
            s.set_tuning(y_tile=tile)
            for phase, nin in ((0, 6), (1, 3)):
                got = s.derivs(phase, torch.from_numpy(f[:nin].astype(np.float32)).cuda()).cpu().numpy()
                for o in range(9):
                    e = np.linalg.norm(got[o] - refs[phase][o]) / np.linalg.norm(refs[phase][o])
                    assert e < 2e-5, (nx, tile, phase, o, e)
        s.close()


@pytest.fixture(scope="module")
def layered384_runs(B):
    nt = 1000
    w = inputs.layered384_workload(nt=nt)
    say("layered384", w.model.shape, nt)
    s = B.Solver.from_workload(w)
    out = {}
    s.set_workload_sources(w)
    out["base"] = s.run(nt).cpu().numpy()[0]
    s.set_sources(w.shot_ofs, w.src_ijk, 2.0 * w.src_m, w.wavelet)
    out["double"] = s.run(nt).cpu().numpy()[0]
    lag = 37
    wl = np.concatenate([np.zeros((1, lag)), w.wavelet[:, :nt - lag]], axis=1)
    s.set_sources(w.shot_ofs, w.src_ijk, w.src_m, wl)
    out["lag"] = s.run(nt).cpu().numpy()[0]
    out["lag_n"] = lag
    s.close()
    return out


def test_layered384_traces_are_finite_and_nonzero(layered384_runs):
    b = layered384_runs["base"]
    assert np.isfinite(b).all()
    for c in range(4):
        assert np.abs(b[c]).max() > 0


def test_layered384_amplitude_scaling_is_exact(layered384_runs):
    np.testing.assert_array_equal(layered384_runs["double"], 2.0 * layered384_runs["base"])


def test_layered384_time_shift_is_exact(layered384_runs):
    lag = layered384_runs["lag_n"]
    a, b = layered384_runs["base"], layered384_runs["lag"]
    assert np.abs(b[..., :lag]).max() == 0.0
    np.testing.assert_array_equal(b[..., lag:], a[..., :-lag])


def test_layered384_one_step_from_a_late_state_matches_oracle(B):
    """Full size, autotuned launch shapes: state after n GPU steps -> one more
    GPU step, against one FP64 oracle step from the same (FP32) state.  The
    tolerance covers the FP32 operators of one step (~1e-6 of each field)."""
    n = 600
    w = inputs.layered384_workload(nt=n + 1)
    say("layered384 one step", w.model.shape, n)
    s = B.Solver.from_workload(w)
    s.set_workload_sources(w)
    s.run(n)
    st = s.get_state()
    tr_gpu = s.run(1).cpu().numpy()[0]
    got = s.get_state()
    lo, hi = s.undamped_range()
    s.close()
    o = oracle.Solver.from_workload(w)
    o.set_sources(w.src_ijk, w.src_m, w.wavelet)
    o.set_state(st.astype(np.float64))
    del st
    o.step = n
    tr_ref = o.run(1)
    ref = o.get_state()
    o.close()
    # the undamped cells keep each field in its first split part
    ref = physics.collapse_undamped(ref, physics.undamped_mask(ref.shape[1:], lo, hi))
    worst = 0.0
    for name, ef, ep in physics.split_errors(got, ref):
        worst = max(worst, ef, ep)
        assert ef <= 2e-5 and ep <= 2e-5, (name, ef, ep)
    for c in range(4):
        e = float(np.linalg.norm(tr_gpu[c] - tr_ref[c]) / np.linalg.norm(tr_ref[c]))
        assert e <= 2e-5, (c, e)
    say(f"  worst field rel-L2 {worst:.2e}")


def test_batch_of_64_shots_matches_single_shots(B):
    nt = 400
    w = inputs.layered128_shots(64, nt=nt)
    say("batch", w.n_shots, nt)
    s = B.Solver.from_workload(w)
    s.set_workload_sources(w)
    batch = s.run(nt).cpu().numpy()
    tuning = s.tuning_values()
    s.close()
    for k in [0, 31, 63]:
        s1 = B.Solver.from_workload(w)
        s1.set_tuning(**tuning)   # the batch's launch shapes: identical arithmetic per shot
        s1.set_sources([0, 1], w.src_ijk[k:k + 1], w.src_m[k:k + 1], w.wavelet[k:k + 1])
        one = s1.run(nt).cpu().numpy()[0]
        s1.close()
        np.testing.assert_array_equal(batch[k], one)


def test_ragged_batch_of_24_models_in_one_graph(B):
    """The 24 uneven models of the ragged batch (64^3 ... 160x160x128, 29 M
    cells in all) advanced together in one graph per step pair equal the same
    models advanced one at a time with the same launch shapes."""
    nt = 100
    ws = inputs.ragged_models(24, nt=nt)
    say("ragged", len(ws), sum(w.cells for w in ws))
    ss = []
    for w in ws:
        s = B.Solver.from_workload(w)
        s.set_workload_sources(w)
        ss.append(s)
    outs = [o.cpu().numpy() for o in B.run_many(ss, nt)]
    for o in outs:
        assert np.isfinite(o).all() and np.abs(o).max() > 0
    for k in [0, 1, 13]:
        w = ws[k]
        s1 = B.Solver.from_workload(w)
        s1.set_tuning(**ss[k].tuning_values())
        s1.set_workload_sources(w)
        np.testing.assert_array_equal(s1.run(nt).cpu().numpy(), outs[k], err_msg=w.name)
        s1.close()
    for s in ss:
        s.close()


def test_run_many_of_uneven_models_against_oracle(B):
    """Three models of uneven size whose lengths are those of the ragged batch
    (80, 96, 120, 144, 160, 48, 64: radix-5, -3 and -2 plans on every axis),
    advanced together by one run_many, against the FP64 oracle run of each
    model alone: the nine fields and each split part (on the scale of its
    field) after nt steps, rel-L2 <= 1e-4 each."""
    nt = 110
    sizes = [(80, 96, 64), (144, 120, 48), (160, 64, 80)]
    ws, ss = [], []
    rng = np.random.default_rng(21)
    for i, (nx, ny, nz) in enumerate(sizes):
        water = max(4, nz // 8)
        m = inputs.layered(nx, ny, nz, water_cells=water, seed=40 + i)
        src = np.array([[nx // 2 + 3, ny // 2 - 2, water + (nz - water) // 2]], np.int32)
        mt = inputs.dc_plus_iso(rng, inputs.DV_UNIT_MOMENT)[None, :]
        # receivers 4 cells above the source: the direct wave reaches them within nt
        sx, sy, sz = (int(v) for v in src[0])
        rec = inputs.receiver_block(sx - 4, sx + 4, sy - 4, sy + 4, sz - 4)
        w = inputs.Workload(f"uneven_{nx}x{ny}x{nz}", m, (10.0, 10.0, 10.0), 0.8e-3, nt, 10, 2.0, 1, 0.0, rec, src,
                            mt, np.array([0, 1], np.int32), inputs.ricker(25.0, 0.8e-3, nt)[None, :])
        ws.append(w)
        s = B.Solver.from_workload(w)
        s.set_workload_sources(w)
        ss.append(s)
    say("run_many uneven", sizes, nt)
    outs = [o.cpu().numpy() for o in B.run_many(ss, nt)]
    for w, s, o in zip(ws, ss, outs):
        got = s.get_state()
        so = oracle.Solver.from_workload(w)
        so.set_sources(w.src_ijk, w.src_m, w.wavelet)
        tr = so.run(nt)
        ref = so.get_state()
        so.close()
        lo, hi = s.undamped_range()
        ref = physics.collapse_undamped(ref, physics.undamped_mask(ref.shape[1:], lo, hi))
        worst = 0.0
        for name, ef, ep in physics.split_errors(got, ref):
            worst = max(worst, ef, ep)
            assert ef <= 1e-4 and ep <= 1e-4, (w.name, name, ef, ep)
        for c in range(4):
            e = float(np.linalg.norm(o[0, c] - tr[c]) / np.linalg.norm(tr[c]))
            assert e <= 1e-4, (w.name, c, e)
        say(f"  {w.name}: worst field rel-L2 {worst:.2e}")
        s.close()


def test_layered384_multistep_against_stored_oracle_planes(B):
    """Full size, in the launch configuration the bench times (one context,
    autotuned shapes, graph replay): the state after the golden's step count
    against the FP64 oracle's on three planes through the source
    (tests/golden/layered384_oracle_planes.npz).  The nine fields (each the sum
    of its split parts) to rel-L2 <= 1e-4; each of the 24 split parts, which
    only the absorbing layer's formulation separates (Sec. II-B), to 1e-4 of
    the norm of the field it sums to."""
    gold = os.path.join(ROOT, "tests", "golden", "layered384_oracle_planes.npz")
    if not os.path.exists(gold):
        pytest.fail("tests/golden/layered384_oracle_planes.npz missing (tests/golden/make_layered384_golden.py writes it)")
    from tests.golden.make_layered128_golden import model_digest
    from tests.golden.make_layered384_golden import planes
    g = np.load(gold, allow_pickle=False)
    nt = int(g["nt"])
    w = inputs.layered384_workload(nt=nt)
    assert str(g["digest"]) == model_digest(w), "workload generator changed since the golden was written"
    say("layered384 multistep", w.model.shape, nt)
    s = B.Solver.from_workload(w)
    s.set_workload_sources(w)
    s.run(nt)
    st = s.get_state()
    mask3 = physics.undamped_mask(w.model.shape, *s.undamped_range())
    s.close()
    for name, zs, ys, xs in planes(w):
        got = st[:, zs, ys, xs].astype(np.float64)
        # the undamped cells keep each field in its first split part
        ref = physics.collapse_undamped(g[name].astype(np.float64), mask3[zs, ys, xs])
        worst_field = worst_part = 0.0
        for fname, parts in SPLIT_PARTS:
            nf = np.linalg.norm(ref[parts].sum(axis=0))
            assert nf > 0, (name, fname)
            e = float(np.linalg.norm(got[parts].sum(axis=0) - ref[parts].sum(axis=0)) / nf)
            worst_field = max(worst_field, e)
            assert e <= 1e-4, (name, fname, e)
            for f in parts:
                ep = float(np.linalg.norm(got[f] - ref[f]) / nf)
                worst_part = max(worst_part, ep)
                assert ep <= 1e-4, (name, oracle.STATE_NAMES[f], ep)
        say(f"  plane {name}: worst field rel-L2 {worst_field:.2e}, worst split part {worst_part:.2e}")


@pytest.mark.parametrize("ny", [16, 75, 144, 240, 384])
def test_derivatives_formed_in_turn_equal_those_of_single_blocks(B, ny):
    """The inverse y kernel gives each derivative a block of its own where the
    launch is small, and otherwise one block per spectrum, which forms both
    derivatives of a spectrum in turn from its tile (at 240 the widest tile
    leaves no room for the symbol in LDS).  A batch of shots takes the second
    form, one shot the first: with every built y tile, two steps of a batch
    from one random state per chosen shot equal those of the shot alone, every
    split part, to FP32 rounding (1e-5 of its largest value, as for every launch
    shape).  The single blocks are checked against the oracle above."""
    import re
    src = open(os.path.join(ROOT, "paper_1705_04874_amd", "csrc", "pstd3d.hip")).read()
    split = int(re.search(r"YINV_SPLIT = (\d+);", src).group(1))
    h, dt, nz = (10.0, 12.0, 9.0), 0.8e-3, 16
    rng = np.random.default_rng(9)
    for nx in (20, 75):
        shape = (nz, ny, nx)
        vp = 2500 + 500 * rng.random(shape)
        args = (vp, vp / 1.8, 310 * vp ** 0.25, h, dt)
        amp = np.where(np.arange(24) < 9, 2e-7, 1.0)[:, None, None, None]
        st = (amp * rng.standard_normal((24,) + shape)).astype(np.float32)
        none = (np.zeros((0, 3)), np.zeros((0, 6)), np.zeros((0, 1)))
        one = B.Solver(*args, pml=4, kspace=1)
        one.set_sources([0, 0], *none)
        batch = B.Solver(*args, pml=4, kspace=1)
        tiles = list(one.tuning()["y_tile_candidates"])
        count = {t: -(-((nx + 1) // 2) // t) + (nx % 2 == 0) for t in tiles}
        shots = split // (6 * nz * min(count.values())) + 1
        for tile in tiles:
            # six spectra in the stress phase, eight in the velocity phase
            assert count[tile] * nz * 8 <= split < count[tile] * nz * 6 * shots
            kw = dict(one.tuning_values(), y_tile=tile)
            one.set_tuning(**kw)
            batch.set_tuning(**kw)
            one.set_sources([0, 0], *none)
            batch.set_sources([0] * (shots + 1), *none)
            one.set_state(st, 0)
            one.run(2)
            ref = one.get_state()
            scale = np.abs(ref).max(axis=(1, 2, 3))
            assert (scale > 0).all()
            chosen = (0, shots // 2, shots - 1)
            for k in chosen:
                batch.set_state(st, 0, shot=k)
            say("in turn", nx, ny, tile, shots)
            batch.run(2)
            for k in chosen:
                err = np.abs(batch.get_state(k) - ref).max(axis=(1, 2, 3))
                assert (err <= 1e-5 * scale).all(), (nx, tile, k, (err / scale).max())
        one.close()
        batch.close()
