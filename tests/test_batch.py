"""Batched stepping: every instance of a batch equals the same instance stepped alone.

The batch runs the single-lattice tile code of every instance inside one launch per
step, so the populations and all three forces of each instance must be bitwise those of
``Sim.step`` with the same call lengths, whatever the schedule (one workgroup per tile or
a persistent grid, direct launches or graph replays, any tile order).  The single path is
itself held to the oracle (test_gpu_parity.py); an FP64 mini batch is also compared with
the oracle directly.
"""
import numpy as np
import pytest

import workloads
from paper_2210_10377_amd.sim import ALL_SCHEMES
from oracle import OracleSim

pytestmark = pytest.mark.gpu

TOL64 = 1e-10


def _members(ws, precision="fp32"):
    from paper_2210_10377_amd import Sim
    return [Sim(w.mask, w.tau, w.uin, precision=precision, box=w.box, max_record=512,
                u_ref=w.u_ref, l_ref=w.l_ref) for w in ws]


def _batch(ws, precision="fp32", max_record=512):
    from paper_2210_10377_amd import Batch
    return Batch(_members(ws, precision), max_record=max_record)


def _seed_states(sims, ws, seed0=100):
    for i, (s, w) in enumerate(zip(sims, ws)):
        S = workloads.near_rest_state(w.nx, w.ny, seed0 + i, amp=0.02, dtype=np.float32)
        s.set_populations(S)


def _singles(ws, calls, precision="fp32", seed0=100):
    """Each instance stepped alone with the given call lengths; (populations, forces)."""
    sims = _members(ws, precision)
    _seed_states(sims, ws, seed0)
    pops, forces = [], []
    for s in sims:
        F = []
        for n in calls:
            s.step(n)
            F.append(s.forces())
        pops.append(s.populations())
        forces.append(np.concatenate(F))
    return pops, forces


def _batched(ws, calls, precision="fp32", schedule=None, seed0=100):
    b = _batch(ws, precision)
    _seed_states(b.members, ws, seed0)
    if schedule:
        b.set_schedule(**schedule)
    F = []
    for n in calls:
        b.step(n)
        Fi, bad = b.forces()
        assert not bad.any()
        F.append(Fi)
    return [m.populations() for m in b.members], np.concatenate(F, axis=1), b


def _assert_same(pa, fa, pb, fb):
    for i in range(len(pa)):
        np.testing.assert_array_equal(pa[i], pb[i], err_msg=f"populations of instance {i}")
        np.testing.assert_array_equal(fa[i], fb[i], err_msg=f"forces of instance {i}")


MINI = workloads.batched_instances(8)
CALLS = (37, 6, 1)

SCHEDULES = {
    "one_block_per_tile": dict(grid_blocks=0, graph_steps=0),
    "persistent_small_grid": dict(grid_blocks=24, graph_steps=0),
    "graph_chunks": dict(grid_blocks=0, graph_steps=8),
    "persistent_graph_shuffled": dict(grid_blocks=40, graph_steps=4, tile_order=12345),
    "tile_queue": dict(grid_blocks=24, graph_steps=0, tile_queue=1),
    "tile_queue_graph_shuffled": dict(grid_blocks=40, graph_steps=4, tile_order=777, tile_queue=1),
    # every instance in one tile shape in the batch (the members keep their own)
    "all_wide_tiles": dict(grid_blocks=0, graph_steps=0, tile_shape="wide"),
    "all_narrow_tiles_graph_shuffled": dict(grid_blocks=0, graph_steps=4, tile_order=99,
                                            tile_shape="narrow"),
    "narrow_tiles_tile_queue": dict(grid_blocks=24, graph_steps=0, tile_queue=1,
                                    tile_shape="narrow"),
}


@pytest.fixture(scope="module")
def mini_singles():
    return _singles(MINI, CALLS)


@pytest.mark.parametrize("name", list(SCHEDULES))
def test_mini_batch_bitwise_equals_singles(name, mini_singles):
    pb, fb, b = _batched(MINI, CALLS, schedule=SCHEDULES[name])
    ps, fs = mini_singles
    _assert_same(ps, [f for f in fs], pb, [fb[i] for i in range(len(MINI))])
    inf = b.info()
    assert inf.steps_done == sum(CALLS)
    for m in b.members:
        assert m.info().steps_done == sum(CALLS)


def test_fp64_mini_batch_against_oracle():
    ws = workloads.batched_instances(4)
    b = _batch(ws, "fp64")
    _seed_states(b.members, ws)
    n = 40
    b.step(n)
    F, bad = b.forces()
    assert not bad.any()
    for i, w in enumerate(ws):
        o = OracleSim(w.mask, w.tau, w.uin, box=w.box)
        o.set_state(workloads.near_rest_state(w.nx, w.ny, 100 + i, amp=0.02, dtype=np.float32))
        o.step(n)
        Fo = o.forces()
        So = o.state()
        Sg = b.members[i].populations()
        fl = w.mask == 0
        assert (np.abs(Sg - So)[:, fl] / np.abs(So)[:, fl]).max() <= TOL64
        for k in range(3):
            scale = np.abs(Fo[:, k]).max()
            assert np.abs(F[i, :, k] - Fo[:, k]).max() / scale <= TOL64, (i, k)


def test_members_changed_between_batch_calls():
    """A member stepped alone, or given a new tau, between batch calls is picked up."""
    ws = MINI[:4]
    b = _batch(ws)
    _seed_states(b.members, ws)
    b.set_schedule(grid_blocks=0, graph_steps=4)
    ref = _members(ws)
    _seed_states(ref, ws)
    b.step(5)
    b.forces()
    for r in ref:
        r.step(5)
        r.forces()
    # instance 1 takes 3 steps alone (its buffers swap parity against the others)
    b.members[1].step(3)
    b.members[1].forces()
    ref[1].step(3)
    ref[1].forces()
    # instance 2 gets a new relaxation time
    b.members[2].set_tau(0.61)
    ref[2].set_tau(0.61)
    b.step(9)
    Fb, _ = b.forces()
    for i, r in enumerate(ref):
        r.step(9)
        np.testing.assert_array_equal(r.forces(), Fb[i])
        np.testing.assert_array_equal(r.populations(), b.members[i].populations())


def test_steps_without_forces_and_ring_overflow():
    from paper_2210_10377_amd import LbmError
    ws = MINI[:3]
    b = _batch(ws, max_record=10)
    _seed_states(b.members, ws)
    ref = _members(ws)
    _seed_states(ref, ws)
    b.set_schedule(grid_blocks=16, graph_steps=6)
    b.step(13, schemes=())
    for r in ref:
        r.step(13, schemes=())
    for i, r in enumerate(ref):
        np.testing.assert_array_equal(r.populations(), b.members[i].populations())
    b.step(10)
    with pytest.raises(LbmError):
        b.step(1)
    F, _ = b.forces()
    assert F.shape == (3, 10, 5, 2)


def test_nonfinite_instance_is_flagged_alone():
    from paper_2210_10377_amd import Sim, Batch
    ws = MINI[:3]
    sims = _members(ws)
    _seed_states(sims, ws)
    # instance 1 starts from a field with a NaN population on a link node
    S = sims[1].populations()
    ys, xs = np.nonzero(ws[1].mask)
    S[1, ys[0], xs[0] - 1] = np.nan
    sims[1].set_populations(S)
    b = Batch(sims, max_record=64)
    b.step(20)
    F, bad = b.forces()
    assert bad.tolist() == [False, True, False]
    assert np.isfinite(F[0]).all() and np.isfinite(F[2]).all()


def test_autotune_keeps_results_bitwise():
    ws = MINI
    b = _batch(ws)
    _seed_states(b.members, ws)
    sched, ms = b.autotune(steps=4)
    assert ms > 0
    assert sched["graph_steps"] in (0, 4)
    assert sched["tile_queue"] in (0, 1) and (sched["grid_blocks"] > 0 or not sched["tile_queue"])
    assert sched["tile_shape"] in ("auto", "wide", "narrow")
    # one block per tile: 2 candidates; 4 persistent grids x (stride, queue) x 2: 16; the
    # fastest with the two other tile shapes: 2
    n_tune = (2 + 16 + 2) * 2 * 4
    assert b.info().steps_done == n_tune
    b.step(7)
    Fb, _ = b.forces()
    ref = _members(ws)
    _seed_states(ref, ws)
    for i, r in enumerate(ref):
        r.step(n_tune, schemes=())
        r.step(7)
        np.testing.assert_array_equal(r.forces(), Fb[i])
        np.testing.assert_array_equal(r.populations(), b.members[i].populations())


def test_full_256_instance_batch_bitwise_equals_singles():
    ws = workloads.batched_instances()
    calls = (10,)
    pb, fb, b = _batched(ws, calls, schedule=dict(grid_blocks=2048, graph_steps=4))
    ps, fs = _singles(ws, calls)
    _assert_same(ps, fs, pb, [fb[i] for i in range(len(ws))])


@pytest.mark.parametrize("precision", ["fp32dev", "fp32sr"])
@pytest.mark.parametrize("collision", ["regularized", "kbc"])
def test_stabilized_collision_batch_bitwise_equals_singles(collision, precision):
    """A batch whose instances all use the regularized or the KBC collision (binary32
    deviations, or binary32 rounded stochastically)."""
    ws = MINI
    from paper_2210_10377_amd import Sim, Batch
    def members():
        return [Sim(w.mask, w.tau, w.uin, precision=precision, box=w.box, max_record=64,
                    collision=collision) for w in ws]
    sims = members()
    _seed_states(sims, ws)
    b = Batch(sims, max_record=64)
    b.set_schedule(grid_blocks=0, graph_steps=4)
    b.step(21)
    Fb, bad = b.forces()
    assert not bad.any()
    ref = members()
    _seed_states(ref, ws)
    for i, r in enumerate(ref):
        r.step(21)
        np.testing.assert_array_equal(r.forces(), Fb[i])
        np.testing.assert_array_equal(r.populations(), b.members[i].populations())


def test_mixed_collision_batch_is_rejected():
    from paper_2210_10377_amd import Sim, Batch, LbmError
    ws = MINI[:2]
    sims = [Sim(w.mask, w.tau, w.uin, precision="fp32", box=w.box, max_record=4,
                collision=c) for w, c in zip(ws, ("bgk", "kbc"))]
    with pytest.raises(LbmError):
        Batch(sims)


@pytest.mark.parametrize("precision", ["fp32", "fp32sr"])
def test_moving_members_batch_bitwise_equals_singles(precision):
    """A batch whose members mix bodies at rest and in rigid motion, with graph replays
    cached before one member starts moving: every instance bitwise equals the same
    member stepped alone with the same motions (binary32 rounded to nearest or
    stochastically)."""
    ws = MINI[:4]
    from paper_2210_10377_amd import Sim, Batch

    def members():
        return [Sim(w.mask, w.tau, w.uin, precision=precision, box=w.box, max_record=64)
                for w in ws]

    def motion(i, phase):
        w = ws[i]
        yc, xc = (np.argwhere(w.mask).mean(axis=0) if w.mask.any() else (0.0, 0.0))
        if i == 1:
            return (0.0, 0.0, 0.002, xc, yc)
        if i == 3 and phase == 1:
            return (0.005, -0.004, -0.001, xc, yc)
        return None

    sims = members()
    _seed_states(sims, ws)
    for i, s in enumerate(sims):
        if motion(i, 0):
            s.set_body_motion(*motion(i, 0))
    b = Batch(sims, max_record=64)
    b.set_schedule(grid_blocks=0, graph_steps=4)
    b.step(9)
    for i, s in enumerate(sims):
        if motion(i, 1):
            s.set_body_motion(*motion(i, 1))
    b.step(9)
    Fb, bad = b.forces()
    assert not bad.any()
    ref = members()
    _seed_states(ref, ws)
    for i, r in enumerate(ref):
        for phase in (0, 1):
            if motion(i, phase):
                r.set_body_motion(*motion(i, phase))
            r.step(9)
        np.testing.assert_array_equal(r.forces(), Fb[i])
        np.testing.assert_array_equal(r.populations(), b.members[i].populations())


@pytest.mark.parametrize("precision", ["fp32", "fp32sr"])
@pytest.mark.parametrize("tile_shape", ["auto", "wide", "narrow"])
def test_member_moving_through_the_grid_batch_bitwise_equals_singles(tile_shape, precision):
    """A member whose body moves one node (and its control volume with it) between two
    batch calls: every instance bitwise equals the same member stepped alone with the
    same calls, also when the batch runs the instances in a tile shape of its own (its
    strip-slot tables follow the member's new plan); a member whose control volume
    changes size stops the batch."""
    from paper_2210_10377_amd import Sim, Batch, LbmError
    ws = MINI[:3]
    k = next(i for i, w in enumerate(ws) if w.box is not None)
    w = ws[k]
    shifted = np.roll(w.mask, 1, axis=1)
    x0, x1, y0, y1 = w.box
    box1 = (x0 + 1, x1 + 1, y0, y1)

    def members():
        return [Sim(v.mask, v.tau, v.uin, precision=precision, box=v.box, max_record=64)
                for v in ws]

    sims = members()
    _seed_states(sims, ws)
    b = Batch(sims, max_record=64)
    b.set_schedule(grid_blocks=0, graph_steps=4, tile_shape=tile_shape)
    b.step(10)
    imp_b = sims[k].set_mask(shifted, box1)
    b.step(10)
    Fb, bad = b.forces()
    assert not bad.any()
    ref = members()
    _seed_states(ref, ws)
    for i, r in enumerate(ref):
        r.step(10)
        if i == k:
            np.testing.assert_array_equal(r.set_mask(shifted, box1), imp_b)
        r.step(10)
        np.testing.assert_array_equal(r.forces(), Fb[i])
        np.testing.assert_array_equal(r.populations(), b.members[i].populations())
    sims[k].set_mask(shifted, (x0 + 1, x1 + 1, y0, y1 - 1))   # one row fewer
    with pytest.raises(LbmError, match="changed size"):
        b.step(1)


def test_batch_mixing_state_layouts_bitwise_equals_singles():
    """Members in the row-interleaved and the planar layout, alternating, in one batch:
    every member bitwise equal to the same member stepped alone."""
    ws = MINI
    from paper_2210_10377_amd import Sim, Batch
    def members():
        return [Sim(w.mask, w.tau, w.uin, precision="fp32", box=w.box, max_record=64,
                    layout=("rows", "planes")[i % 2]) for i, w in enumerate(ws)]
    sims = members()
    _seed_states(sims, ws)
    b = Batch(sims, max_record=64)
    b.set_schedule(grid_blocks=24, graph_steps=4)
    b.step(21)
    Fb, bad = b.forces()
    assert not bad.any()
    ref = members()
    _seed_states(ref, ws)
    for i, r in enumerate(ref):
        r.step(21)
        np.testing.assert_array_equal(r.forces(), Fb[i])
        np.testing.assert_array_equal(r.populations(), b.members[i].populations())


def test_schedule_validation():
    """A tile queue needs a persistent grid; tile_queue takes 0 or 1."""
    from paper_2210_10377_amd import LbmError
    b = _batch(MINI[:2])
    with pytest.raises(LbmError):
        b.set_schedule(grid_blocks=0, tile_queue=1)
    with pytest.raises(LbmError):
        b.set_schedule(grid_blocks=16, tile_queue=2)
    b.set_schedule(grid_blocks=16, tile_queue=1)
    assert b.info().schedule.tile_queue == 1
    # tile_shape takes LBM_TILE_AUTO, LBM_TILE_WIDE or LBM_TILE_NARROW
    import ctypes
    from paper_2210_10377_amd import _capi as C
    s = C.lbm_batch_schedule(0, 0, 0, 0, 7)
    assert C.load().lbm_batch_set_schedule(b._h, ctypes.byref(s)) == C.LBM_EINVAL
    b.set_schedule(tile_shape="narrow")
    assert b.info().schedule.tile_shape == C.LBM_TILE_NARROW


@pytest.mark.gpu
@pytest.mark.parametrize("precision", ["fp64", "fp32dev"])
def test_fused_batch_bitwise_equals_singles(precision):
    """A batch large enough for three steps per launch, among its members one in motion and one
    moved through the grid between the calls: every instance bitwise equal to the member
    stepped alone (whatever launches each takes), in calls of 1, 8 and 3 steps."""
    from paper_2210_10377_amd import Batch, Sim
    ws = workloads.batched_instances(14, seed=11)
    runs = []
    for batched in (True, False):
        sims = [Sim(w.mask, w.tau, w.uin, precision=precision, box=w.box, max_record=12,
                    u_ref=w.u_ref, l_ref=w.l_ref) for w in ws]
        assert sum(s.nx * s.ny for s in sims) >= 400_000
        sims[3].set_body_motion(ux=0.004, omega=1e-4, xc=0.3 * sims[3].nx, yc=0.5 * sims[3].ny)
        b = Batch(sims, max_record=12) if batched else None
        out = []
        for k in (1, 8, 3):
            print(f"fused batch {precision} batched={batched} k={k}", flush=True)
            if batched:
                b.step(k)
                F = list(b.forces()[0])
            else:
                for s in sims:
                    s.step(k)
                F = [s.forces() for s in sims]
            out.append(F)
            if k == 8:
                m = np.roll(ws[5].mask, 1, axis=1)
                box = (ws[5].box[0] + 1, ws[5].box[1] + 1, *ws[5].box[2:])
                out.append([sims[5].set_mask(m, box)])
        out.append([s.populations() for s in sims])
        runs.append(out)
        del b, sims
    for a, c in zip(*runs):
        for x, y in zip(a, c):
            np.testing.assert_array_equal(x, y)


@pytest.mark.gpu
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_batch_with_tiled_body_rectangles_bitwise_equals_singles(precision):
    """Above 1e6 nodes the body rectangles of a batch take a launch of tiles with forces:
    every instance bitwise equal to the member stepped alone, in calls of 4 and 3 steps."""
    from paper_2210_10377_amd import Batch, Sim
    ws = workloads.batched_instances(28, seed=13)
    runs = []
    for batched in (True, False):
        sims = [Sim(w.mask, w.tau, w.uin, precision=precision, box=w.box, max_record=8,
                    u_ref=w.u_ref, l_ref=w.l_ref) for w in ws]
        assert sum(s.nx * s.ny for s in sims) >= 1_000_000
        b = Batch(sims, max_record=8) if batched else None
        out = []
        for k in (4, 3):
            print(f"tiled batch {precision} batched={batched} k={k}", flush=True)
            if batched:
                b.step(k)
                out.append(list(b.forces()[0]))
            else:
                for s in sims:
                    s.step(k)
                out.append([s.forces() for s in sims])
        out.append([s.populations() for s in sims])
        runs.append(out)
        del b, sims
    for a, c in zip(*runs):
        for x, y in zip(a, c):
            np.testing.assert_array_equal(x, y)


@pytest.mark.gpu
def test_batch_whose_bodies_take_all_of_the_lattices():
    """Control volumes that span the lattices: every node is in a body rectangle, so launches of
    three steps would be launches of body windows alone.  Members bitwise equal to lattices
    stepped alone, in calls of 3 and 4 steps."""
    from paper_2210_10377_amd import Batch, Sim
    nx, ny, n = 512, 256, 60
    mask = np.zeros((ny, nx), np.uint8)
    mask[120:130, 150:165] = 1
    box = (1, nx - 1, 1, ny - 1)
    rng = np.random.default_rng(17)
    uin = [0.05 * (1 + 0.1 * rng.uniform(-1, 1, ny)) for _ in range(n)]

    def member(i):
        return Sim(mask, 0.6 + 0.002 * i, uin[i], precision="fp64", box=box, max_record=8)

    sims = [member(i) for i in range(n)]
    b = Batch(sims, max_record=8)
    F = []
    for k in (3, 4):
        print(f"batch of whole lattices k={k}", flush=True)
        b.step(k)
        F.append(b.forces()[0])
    for i in (0, 31, n - 1):
        alone = member(i)
        for k, f in zip((3, 4), F):
            alone.step(k)
            np.testing.assert_array_equal(f[i], alone.forces())
        np.testing.assert_array_equal(sims[i].populations(), alone.populations())


@pytest.mark.gpu
@pytest.mark.parametrize("schemes", [ALL_SCHEMES, ()])
def test_autotune_times_what_the_schedule_governs(schemes):
    """In a batch that takes three steps a launch the candidates are timed on launches of one
    step: the others are the same whatever the schedule.  Results stay those of 40 x 9 steps."""
    from paper_2210_10377_amd import Batch
    ws = workloads.batched_instances(28, seed=13)
    b = Batch.from_workloads(ws, precision="fp64", max_record=24)
    b.step(7, schemes)
    assert b.launches() == (1, 2)
    _, ms = b.autotune(steps=9, schemes=() if not schemes else ("A",))
    assert b.launches() == (1 + 40 * 9, 2) and ms > 0
    b.step(6, schemes)
    assert b.launches() == (1 + 40 * 9, 4)
    assert b.info().steps_done == 7 + 40 * 9 + 6
    for i in (0, 13, 27):
        alone = Batch.from_workloads([ws[i]], precision="fp64", max_record=12).members[0]
        alone.step(7 + 40 * 9 + 6, schemes=())
        np.testing.assert_array_equal(b.members[i].populations(), alone.populations())


@pytest.mark.gpu
def test_motion_that_begins_in_a_batch_brings_launches_of_three_steps():
    """Binary32 lattices of which single steps are the faster form at rest and launches of three
    steps with a body in motion: each takes its form, from the call after the change on, back again
    too, and the members stay bitwise equal to lattices stepped alone."""
    from paper_2210_10377_amd import Batch, Sim
    nx, ny, n = 200, 80, 62
    mask = np.zeros((ny, nx), np.uint8)
    mask[40:66, 50:76] = 1
    box = (48, 78, 38, 68)
    rng = np.random.default_rng(29)
    uin = [0.05 * (1 + 0.1 * rng.uniform(-1, 1, ny)) for _ in range(n)]

    def member(i):
        return Sim(mask, 0.6 + 0.002 * i, uin[i], precision="fp32", box=box, max_record=8)

    def spin(sim, omega):
        sim.set_body_motion(omega=omega, xc=63.0, yc=53.0)

    sims = [member(i) for i in range(n)]
    b = Batch(sims, max_record=8)
    F, forms = [], []
    for omega in (0.0, 1e-4, 0.0):
        print(f"batch motion omega={omega}", flush=True)
        spin(sims[5], omega)
        b.step(7)
        F.append(b.forces()[0])
        forms.append(b.launches())
    assert forms == [(7, 0), (8, 2), (15, 2)]
    for i in (0, 5, n - 1):
        alone = member(i)
        for omega, f in zip((0.0, 1e-4, 0.0), F):
            if i == 5:
                spin(alone, omega)
            alone.step(7)
            np.testing.assert_array_equal(f[i], alone.forces())
        np.testing.assert_array_equal(sims[i].populations(), alone.populations())


@pytest.fixture(scope="module")
def few_singles():
    return _singles(MINI[:4], CALLS)


@pytest.mark.parametrize("name", list(SCHEDULES))
def test_schedules_of_a_batch_of_single_steps(name, few_singles):
    """Every schedule on a batch that takes all of its steps in launches of one step, replaying
    whole graphs and reducing each row in the launch after it."""
    ws = MINI[:4]
    b = _batch(ws)
    _seed_states(b.members, ws)
    b.set_schedule(**SCHEDULES[name])
    F = []
    for n in CALLS:
        b.step(n)
        Fi, bad = b.forces()
        assert not bad.any()
        F.append(Fi)
    assert b.launches() == (sum(CALLS), 0)
    F = np.concatenate(F, axis=1)
    ps, fs = few_singles
    _assert_same(ps, fs, [m.populations() for m in b.members], [F[i] for i in range(len(ws))])


def test_many_members_of_single_steps_with_a_persistent_schedule():
    """Sixty-four lattices rounded stochastically, which take single steps: a persistent grid,
    graphs of four launches and a shuffled list."""
    ws = workloads.batched_instances(64)
    from paper_2210_10377_amd import Batch
    b = Batch.from_workloads(ws, precision="fp32sr", max_record=16)
    b.set_schedule(grid_blocks=1024, graph_steps=4, tile_order=7)
    b.step(10)
    F, bad = b.forces()
    assert not bad.any() and b.launches() == (10, 0)
    for i in (0, 17, 40, 63):
        r = _members([ws[i]], "fp32sr")[0]
        r.step(10)
        np.testing.assert_array_equal(r.forces(), F[i])
        np.testing.assert_array_equal(r.populations(), b.members[i].populations())


def _box_around(mask, grow):
    ys, xs = np.nonzero(mask.any(1))[0], np.nonzero(mask.any(0))[0]
    return int(xs[0]) - grow, int(xs[-1]) + 1 + grow, int(ys[0]) - grow, int(ys[-1]) + 1 + grow


def _odd_members(precision):
    """Lattices of all kinds and boundaries in one batch: two that make launches of three steps
    worth taking, and narrow, thin, tiny and full ones."""
    from paper_2210_10377_amd import Sim
    rng = np.random.default_rng(23)
    sims = []
    shapes = [(900, 700), (251, 300), (203, 201), (500, 3), (3, 400), (37, 300), (5, 5), (64, 64), (65, 90),
              (130, 17), (111, 130), (200, 120), (1501, 803)]
    for i, (nx, ny) in enumerate(shapes):
        mask = np.zeros((ny, nx), np.uint8)
        box, bc = None, (0, 0)
        if i == 0:
            mask[300:330, 200:260] = 1
            box = _box_around(mask, 20)
        elif i == 1:  # at the outlet, at a wall and across the wrap
            mask[100:120, nx - 1] = 1
            mask[0:3, 90:100] = 1
            bc = (0, 1)
        elif i == 2:
            mask[5:9, 0:2] = 1
            bc = (1, 0)
        elif i == 8:
            mask[20:25, 30:34] = 1
            box = (1, nx - 1, 1, ny - 1)  # every node has force terms
        elif i == 10:  # scattered solids
            mask[4:-4, 4:-4] = rng.uniform(size=(ny - 8, nx - 8)) < 0.05
            bc = (1, 1)
        elif min(nx, ny) >= 17:
            mask[ny // 2:ny // 2 + 3, nx // 3:nx // 3 + 4] = 1
            box = _box_around(mask, 2)
        uin = 0.05 * (1 + 0.1 * rng.uniform(-1, 1, ny))
        s = Sim(mask, 0.55 + 0.01 * i, uin, precision=precision, bc_x=bc[0], bc_y=bc[1], box=box, max_record=16)
        s.set_populations(workloads.NEAR_REST_BASE[:, None, None] * (
            1 + 0.02 * rng.uniform(-1, 1, (9, ny, 1)) * rng.uniform(-1, 1, (9, 1, nx))))
        if i in (0, 11):
            s.set_body_motion(ux=0.004, omega=1e-4, xc=nx / 3, yc=ny / 2)
        sims.append(s)
    return sims


@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp32dev"])
@pytest.mark.parametrize("schemes", [ALL_SCHEMES, ()])
def test_odd_members_in_launches_of_three_steps(precision, schemes):
    """Every member bitwise equal to itself in single steps (DRTT of a call's last step to the
    rounding of the sum over its box)."""
    from paper_2210_10377_amd import Batch
    sims, ref = _odd_members(precision), _odd_members(precision)
    b = Batch(sims, max_record=16)
    b.step(7, schemes)
    assert b.launches() == (1, 2)
    F = b.forces()[0] if schemes else None
    for i, (s, r) in enumerate(zip(sims, ref)):
        for n in (2, 2, 2, 1):
            r.step(n, schemes)
        np.testing.assert_array_equal(s.populations(), r.populations(), err_msg=f"member {i}")
        if schemes:
            Fr = r.forces()
            np.testing.assert_array_equal(F[i][:, [0, 1, 3]], Fr[:, [0, 1, 3]], err_msg=f"member {i}")
            if i in (0, 8):
                box = (1, 64, 1, 89) if i == 8 else (180, 280, 280, 350)
                N = (box[1] - box[0]) * (box[3] - box[2]) * 9
                assert np.abs(F[i] - Fr).max() <= 4 * N * 0.45 * 2.0 ** -53


@pytest.mark.parametrize("precision,nx,ny", [("fp32sr", 2803, 801), ("fp16dev", 3003, 2001)])
def test_large_members_of_the_other_storages_in_launches_of_three_steps(precision, nx, ny):
    """Stochastically rounded and binary16 lattices large enough for launches of three steps, one
    with a control volume of 1.2e5 nodes (which takes tiles with forces), without forces and with
    them: bitwise those of single steps."""
    from paper_2210_10377_amd import Batch, Sim

    def members():
        rng = np.random.default_rng(29)
        sims = []
        for i in range(3):
            mask = np.zeros((ny, nx), np.uint8)
            mask[ny // 2 - 20:ny // 2 + 20, 600:660] = 1
            box = (500, 900, ny // 2 - 150, ny // 2 + 150) if i == 0 else (590, 670, ny // 2 - 30, ny // 2 + 30)
            s = Sim(mask, 0.55 + 0.01 * i, np.full(ny, 0.05), precision=precision, box=box, max_record=8)
            if i < 2:
                s.set_populations(workloads.NEAR_REST_BASE[:, None, None] * (
                    1 + 0.02 * rng.uniform(-1, 1, (9, ny, 1)) * rng.uniform(-1, 1, (9, 1, nx))))
            sims.append(s)
        return sims

    sims, ref = members(), members()
    b = Batch(sims, max_record=8)
    b.step(4, ())
    print(f"large members {precision}: without forces", flush=True)
    b.step(3, ALL_SCHEMES)
    print(f"large members {precision}: with forces", flush=True)
    assert b.launches() == (1, 2)
    F = b.forces()[0]
    for i, (s, r) in enumerate(zip(sims, ref)):
        for n, sch in ((2, ()), (2, ()), (2, ALL_SCHEMES), (1, ALL_SCHEMES)):
            r.step(n, sch)
        np.testing.assert_array_equal(F[i][:, [0, 1, 3]], r.forces()[:, [0, 1, 3]], err_msg=f"member {i}")
        np.testing.assert_array_equal(s.populations(), r.populations(), err_msg=f"member {i}")


def _captured_launches(stream, call):
    """Kernel launches that `call` enqueues on a stream (by capturing them; they are not run)."""
    import ctypes
    import torch
    hip = ctypes.CDLL("libamdhip64.so")
    st = ctypes.c_void_p(stream.cuda_stream)
    graph, n = ctypes.c_void_p(), ctypes.c_size_t()
    torch.cuda.synchronize()
    assert hip.hipStreamBeginCapture(st, 1) == 0
    try:
        call()
    finally:
        rc = hip.hipStreamEndCapture(st, ctypes.byref(graph))
    assert rc == 0 and hip.hipGraphGetNodes(graph, None, ctypes.byref(n)) == 0
    hip.hipGraphDestroy(graph)
    return n.value


def test_calls_without_single_steps_do_not_reset_the_tile_queue():
    """The tile queue belongs to launches of one step: a call that takes none enqueues the
    launches of three steps alone."""
    import torch
    from paper_2210_10377_amd import Batch
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        b = Batch.from_workloads(workloads.batched_instances(28, seed=13), precision="fp64", max_record=8,
                                 stream=st)
        b.set_schedule(grid_blocks=256, tile_queue=1)
        b.step(4, ())
        assert b.launches() == (1, 1)
        # (A step by the schedule comes with the reset of the queue.)
        assert _captured_launches(st, lambda: b.step(6, ())) == 2
        assert _captured_launches(st, lambda: b.step(4, ())) == 3
