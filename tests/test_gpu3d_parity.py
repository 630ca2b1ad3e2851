"""GPU parity of the three-dimensional (D3Q27) HIP path against the 3-D oracle, both fed
from the same seeded inputs.  FP64: populations and every force within 1e-10 of the
oracle (relative).  32-bit storage: forces within 1e-4 of the largest force of the run
(DRTT of random fields: 1e-2, the rounding of the box momenta).  FP16 deviations: 5e-2."""
import numpy as np
import pytest

import workloads
from oracle import d3q27 as D
from workloads import d3

pytestmark = pytest.mark.gpu

TOL64 = 1e-10


def _sim3(mask, tau, uin=None, **kw):
    from paper_2210_10377_amd import Sim3
    return Sim3(mask, tau, uin, **kw)


def _pop_err(Sg, So, mask):
    fl = mask == 0
    return (np.abs(Sg - So)[:, fl] / np.abs(So)[:, fl]).max()


def _force_err(Fg, Fo, cols=(0, 1, 2, 3)):
    out = []
    for k in cols:
        scale = np.abs(Fo[:, k]).max()
        assert scale > 0, k
        out.append(np.abs(Fg[:, k] - Fo[:, k]).max() / scale)
    return np.array(out)


def _edge_mask():
    m = np.zeros((10, 12, 70), np.uint8)
    m[2:4, 3:5, 66:70] = 1      # touches the outlet plane
    m[0, 4:6, 20:23] = 1        # on a z wall
    m[5:7, 0:2, 0:2] = 1        # on the inlet plane and a y wall
    m[6, 6, 40] = 1             # single node
    return m


CASES = {
    # name: (mask builder, bc (x, y, z), box, inlet speed)
    "sphere_walls_box": (lambda: d3.sphere_mask(40, 24, 22, 14, 11.5, 10.5, 5),
                         (0, 0, 0), (6, 23, 4, 20, 3, 19), 0.04),
    "sphere_periodic_box": (lambda: d3.sphere_mask(36, 20, 18, 17, 9.5, 8.5, 4.5),
                            (1, 1, 1), (10, 25, 3, 17, 2, 16), None),
    "extruded_periodic_span": (lambda: d3.extrude(workloads.cylinder_mask(50, 22, 16, 10.5, 4), 6),
                               (0, 0, 1), (8, 25, 3, 19, 0, 6), 0.04),
    "edges_no_box": (_edge_mask, (0, 0, 0), None, 0.03),
    "multi_tile_ragged": (lambda: d3.sphere_mask(300, 18, 14, 100, 8.5, 6.5, 4),
                          (0, 1, 0), (90, 111, 2, 16, 1, 13), 0.05),
}


@pytest.mark.parametrize("name", list(CASES))
def test_fp64_small_cases_random_state(name):
    """Every boundary rule in three dimensions, alone and together, from a seeded random
    near-rest state, 40 steps, FP64: populations and all four forces to 1e-10."""
    mk, (bx, by, bz), box, u = CASES[name]
    mask = mk()
    nz, ny, nx = mask.shape
    uin = None if bx == 1 else np.linspace(0.5, 1.0, ny)[None, :] * np.linspace(1.0, 0.8, nz)[:, None] * u
    S0 = d3.near_rest_state3(nx, ny, nz, seed=len(name), amp=0.05)
    o = D.OracleSim3(mask, tau=0.7, uin=uin, bc_x=bx, bc_y=by, bc_z=bz, box=box)
    o.set_state(S0)
    o.step(40)
    g = _sim3(mask, 0.7, uin, precision="fp64", bc_x=bx, bc_y=by, bc_z=bz, box=box,
              max_record=64)
    g.set_populations(S0)
    g.step(40)
    Fg, Fo = g.forces(), o.forces()
    assert Fg.shape == Fo.shape == (40, 4, 3)
    assert _pop_err(g.populations(), o.state(), mask) <= TOL64
    cols = (0, 1, 2, 3) if box is not None else (0, 1, 3)
    e = _force_err(Fg, Fo, cols)
    assert np.all(e <= TOL64), e
    if box is None:
        assert np.all(np.isnan(Fg[:, 2]))


@pytest.fixture(scope="module")
def sphere_reference():
    w = d3.sphere_channel_64x32x32()
    o = D.OracleSim3(w.mask, tau=w.tau, uin=w.uin, box=w.box)
    o.step(w.steps)
    return w, o.state(), o.forces()


@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp32dev", "fp32sr", "fp16dev"])
def test_sphere_channel_from_rest(precision, sphere_reference):
    """Sphere (D = 10) in a walled duct at Re 20, 300 steps from rest: FP64 populations
    and forces to 1e-10; 32-bit storage forces to 1e-4 (DRTT 1e-3), FP16 deviations
    5e-2; DRTT equals MEA-B in FP64; symmetric sphere: side forces vanish."""
    w, So, Fo = sphere_reference
    g = _sim3(w.mask, w.tau, w.uin, precision=precision, box=w.box, max_record=300)
    Fg = g.run(w.steps)
    assert np.isfinite(Fg).all()
    e = _force_err(Fg, Fo)
    print(precision, "sphere force errors (A, B, DRTT, SI):", e)
    tol = {"fp64": np.full(4, TOL64), "fp32": np.array([1e-4, 1e-4, 1e-3, 1e-4]),
           "fp32dev": np.array([1e-4, 1e-4, 1e-3, 1e-4]),
           "fp32sr": np.array([1e-4, 1e-4, 1e-3, 1e-4]),
           "fp16dev": np.full(4, 5e-2)}[precision]
    assert np.all(e <= tol), e
    if precision == "fp64":
        assert _pop_err(g.populations(), So, w.mask) <= TOL64
        sc = np.abs(Fg[:, 1]).max()
        assert np.abs(Fg[:, 2] - Fg[:, 1]).max() <= 1e-9 * sc


def test_deterministic_bitwise_and_chunked_calls():
    """Two runs give identical populations and forces; 30 steps in one call equal
    30 steps in calls of 7, 1, 22 (the force rows included)."""
    w = d3.sphere_channel_64x32x32()
    outs = []
    for calls in ((30,), (30,), (7, 1, 22)):
        g = _sim3(w.mask, w.tau, w.uin, precision="fp32", box=w.box, max_record=64)
        F = []
        for n in calls:
            g.step(n)
            F.append(g.forces())
        outs.append((g.populations(), np.concatenate(F)))
    for p, f in outs[1:]:
        assert np.array_equal(outs[0][0], p)
        assert np.array_equal(outs[0][1], f, equal_nan=True)


def test_forces_off_same_populations_and_scheme_selection():
    w = d3.sphere_channel_64x32x32()
    g1 = _sim3(w.mask, w.tau, w.uin, precision="fp64", box=w.box, max_record=50)
    g2 = _sim3(w.mask, w.tau, w.uin, precision="fp64", box=w.box, max_record=50)
    g1.step(20, schemes=())
    g2.step(20, schemes=("B",))
    assert np.array_equal(g1.populations(), g2.populations())
    assert g1.forces().shape == (0, 4, 3)
    F = g2.forces()
    assert np.all(np.isnan(F[:, [0, 2, 3]])) and np.all(np.isfinite(F[:, 1]))


@pytest.mark.parametrize("precision", ["fp32", "fp32sr", "fp64"])
def test_full_size_naca3d_two_steps(precision):
    """The benchmark's 3-D airfoil (1920 x 192 x 96, periodic span, box over the whole
    span) in its launch configuration, FP32 and FP64, from a seeded random state: every
    fluid population and every force row of two steps against the oracle."""
    w = d3.naca3d(24, 200.0)
    S0 = d3.near_rest_state3(w.nx, w.ny, w.nz, seed=5, amp=0.02,
                             dtype=np.float64 if precision == "fp64" else np.float32)
    g = _sim3(w.mask, w.tau, w.uin, precision=precision, bc_z=w.bc_z, box=w.box, max_record=4)
    g.set_populations(S0)
    g.step(2)
    Fg, Sg = g.forces(), g.populations()
    del g
    o = D.OracleSim3(w.mask, tau=w.tau, uin=w.uin, bc_z=w.bc_z, box=w.box)
    o.set_state(S0)
    del S0
    o.step(2)
    Fo = o.forces()
    So = o.state()
    del o
    fl = w.mask == 0
    err = 0.0
    for i in range(27):
        err = max(err, float((np.abs(Sg[i] - So[i])[fl] / So[i][fl]).max()))
    # binary32 rounding of the collision relative to the smallest populations (corner
    # weight 1/216, six times below the smallest D2Q9 weight); stochastic rounding stores
    # either neighbour, up to one unit in the last place instead of half of one
    assert err <= {"fp32": 1e-5, "fp32sr": 2e-5, "fp64": TOL64}[precision], err
    e = _force_err(Fg, Fo)
    print("full-size 3-D population error", err, "force errors", e)
    # A random field's forces are sums of random link terms: binary32 rounding of the
    # populations (2.4e-6 relative, above) summed over the ~4e4 links of the span moves
    # A and B by about 1e-4 of the largest force (measured 7e-5 .. 1.1e-4).
    tol = np.full(4, TOL64) if precision == "fp64" else np.array([2e-4, 2e-4, 1e-2, 1e-3])
    assert np.all(e <= tol), e


def test_ring_overflow_zero_steps_and_bad_arguments():
    """The ring refuses steps it cannot hold (nothing enqueued), zero steps do nothing,
    unknown scheme bits and negative counts are refused; the state is unchanged by the
    refusals."""
    from paper_2210_10377_amd import LbmError
    w = d3.sphere_channel_64x32x32()
    g = _sim3(w.mask, w.tau, w.uin, precision="fp32", box=w.box, max_record=8)
    g.step(5)
    before = g.populations()
    with pytest.raises(LbmError, match="overflow"):
        g.step(4)
    g.step(0)
    g.step(1, schemes=())  # no force row: allowed with the ring nearly full
    assert g.info().steps_done == 6
    L = g._lib
    assert L.lbm3d_step(g._h, 1, 1 << 7) == -1
    assert L.lbm3d_step(g._h, -1, 15) == -1
    F = g.forces()
    assert F.shape == (5, 4, 3) and np.isfinite(F).all()
    g2 = _sim3(w.mask, w.tau, w.uin, precision="fp32", box=w.box, max_record=8)
    g2.step(5)
    g2.forces()
    g2.step(1, schemes=())
    assert np.array_equal(g.populations(), g2.populations())
    del before


def test_nonfinite_state_is_reported():
    """A NaN planted in the state reaches the forces: lbm3d_forces reports it
    (LBM_ENONFINITE) and still returns the rows."""
    w = d3.sphere_channel_64x32x32()
    g = _sim3(w.mask, w.tau, w.uin, precision="fp64", box=w.box, max_record=8)
    S = g.populations()
    x0, x1, y0, y1, z0, z1 = w.box
    S[3, (z0 + z1) // 2, y0 + 1, x0 + 1] = np.nan
    g.set_populations(S)
    g.step(3)
    F = g.forces()
    assert g.last_nonfinite and F.shape == (3, 4, 3)
    assert not np.isfinite(F[:, 2]).all()


@pytest.mark.parametrize("name", ["sphere_walls_box", "extruded_periodic_span", "edges_no_box"])
def test_fp64_regularized_small_cases(name):
    """The regularized collision (for tau_lb near 1/2) at tau_lb 0.505 from a random
    near-rest state, 40 steps, FP64: populations and forces to 1e-10 of the oracle."""
    mk, (bx, by, bz), box, u = CASES[name]
    mask = mk()
    nz, ny, nx = mask.shape
    uin = None if bx == 1 else np.full((nz, ny), u)
    S0 = d3.near_rest_state3(nx, ny, nz, seed=40 + len(name), amp=0.05)
    o = D.OracleSim3(mask, tau=0.505, uin=uin, bc_x=bx, bc_y=by, bc_z=bz, box=box,
                     collision="regularized")
    o.set_state(S0)
    o.step(40)
    g = _sim3(mask, 0.505, uin, precision="fp64", bc_x=bx, bc_y=by, bc_z=bz, box=box,
              max_record=64, collision="regularized")
    g.set_populations(S0)
    g.step(40)
    assert _pop_err(g.populations(), o.state(), mask) <= TOL64
    cols = (0, 1, 2, 3) if box is not None else (0, 1, 3)
    e = _force_err(g.forces(), o.forces(), cols)
    assert np.all(e <= TOL64), e


@pytest.mark.parametrize("precision", ["fp64", "fp32dev", "fp32sr"])
def test_regularized_sphere_low_viscosity(precision):
    """The sphere duct at tau_lb 0.506 (Re 200 on the diameter) with the regularized
    collision, 300 steps from rest: FP64 forces to 1e-10 of the oracle, binary32 deviations
    and binary32 rounded stochastically to 1e-3 (relative to the largest force)."""
    w = d3.sphere_channel_64x32x32()
    tau = 0.506
    o = D.OracleSim3(w.mask, tau=tau, uin=w.uin, box=w.box, collision="regularized")
    o.step(300)
    Fo = o.forces()
    g = _sim3(w.mask, tau, w.uin, precision=precision, box=w.box, max_record=300,
              collision="regularized")
    Fg = g.run(300)
    assert np.isfinite(Fg).all()
    e = _force_err(Fg, Fo)
    assert np.all(e <= (TOL64 if precision == "fp64" else 1e-3)), e


@pytest.mark.parametrize("precision,name", [("fp32", "sphere_walls_box"),
                                            ("fp16dev", "multi_tile_ragged"),
                                            ("fp32sr", "multi_tile_ragged"),
                                            ("fp64", "extruded_periodic_span")])
def test_row_interleaved_and_planar_layouts_agree_bitwise(precision, name):
    """The two device layouts of the state run the same arithmetic: populations and
    forces bitwise equal after 30 steps from a random state."""
    mk, (bx, by, bz), box, u = CASES[name]
    mask = mk()
    nz, ny, nx = mask.shape
    uin = None if bx == 1 else np.full((nz, ny), u)
    S0 = d3.near_rest_state3(nx, ny, nz, seed=70, amp=0.05)
    runs = []
    for layout in ("rows", "planes"):
        g = _sim3(mask, 0.7, uin, precision=precision, bc_x=bx, bc_y=by, bc_z=bz, box=box,
                  max_record=64, layout=layout)
        g.set_populations(S0)
        g.step(30)
        runs.append((g.populations(), g.forces()))
    np.testing.assert_array_equal(runs[0][0], runs[1][0])
    np.testing.assert_array_equal(runs[0][1], runs[1][1])


def test_checkpoint_reset_and_parameter_changes_3d():
    """2n steps equal n steps, a checkpoint, a new handle restoring it, n steps (bitwise,
    populations and forces); a checkpoint of the other layout is refused; reset equals a
    fresh handle; set_tau and set_inlet between calls equal a handle created with the new
    values and restored from the checkpoint (FP32 sphere duct)."""
    from paper_2210_10377_amd import LbmError
    w = d3.sphere_channel_64x32x32()
    mk = lambda tau=w.tau, uin=w.uin, layout="auto": _sim3(
        w.mask, tau, uin, precision="fp32", box=w.box, max_record=64, layout=layout)
    a = mk()
    a.step(40)
    Fa = a.forces()
    b = mk()
    b.step(20)
    Fb = b.forces()
    blob = b.get_state()
    c = mk()
    c.set_state(blob)
    c.step(20)
    assert np.array_equal(a.populations(), c.populations())
    assert np.array_equal(Fa, np.concatenate([Fb, c.forces()]))
    assert c.info().steps_done == 40
    with pytest.raises(LbmError):
        mk(layout="planes").set_state(blob)
    c.reset()
    c.step(20)
    f = mk()
    f.step(20)
    assert np.array_equal(c.populations(), f.populations())
    assert np.array_equal(c.forces(), f.forces())
    # parameter changes between calls
    tau2, uin2 = w.tau * 1.1, np.asarray(w.uin) * 0.8
    b.set_tau(tau2)
    b.set_inlet(uin2)
    b.step(20)
    d = mk(tau=tau2, uin=uin2)
    d.set_state(blob)
    d.step(20)
    assert np.array_equal(b.populations(), d.populations())
    assert np.array_equal(b.forces(), d.forces())


@pytest.mark.parametrize("precision,shape", [("fp32sr", (200, 71, 70)), ("fp32sr", (201, 72, 70)),
                                             ("fp16dev", (130, 55, 55)), ("fp16dev", (130, 56, 56)),
                                             ("fp32", (130, 56, 56)), ("fp64", (201, 72, 70))])
def test_force_strips_joined_and_apart(precision, shape):
    """Grids on both sides of the sizes where the strips with force terms leave the step's
    launch (1e6 nodes stochastically rounded, 4e5 in binary16), and others that never do:
    two steps of a random state with forces against the oracle, populations bitwise those of
    steps without forces.  Tolerances as for the large airfoil above; binary16 5e-2 (its
    rounding of 5e-4 of a deviation, over the box of about 1e4 nodes against a force of random
    terms over about 1e3 links)."""
    nx, ny, nz = shape
    mask = d3.sphere_mask(nx, ny, nz, 0.3 * nx, ny / 2, nz / 2, 6.3)
    c = (int(0.3 * nx), ny // 2, nz // 2)
    box = tuple(v for m in c for v in (m - 10, m + 11))
    S0 = d3.near_rest_state3(nx, ny, nz, seed=7, amp=0.02,
                             dtype=np.float64 if precision == "fp64" else np.float32)
    sims = [_sim3(mask, 0.56, 0.04, precision=precision, box=box, max_record=4) for _ in range(2)]
    for g, schemes in zip(sims, (None, ())):
        g.set_populations(S0)
        g.step(2, **({} if schemes is None else {"schemes": schemes}))
    Fg = sims[0].forces()
    np.testing.assert_array_equal(sims[0].populations(), sims[1].populations())
    o = D.OracleSim3(mask, tau=0.56, uin=np.full((nz, ny), 0.04), box=box)
    o.set_state(S0)
    o.step(2)
    e = _force_err(Fg, o.forces())
    print(precision, shape, "force errors", e)
    tol = {"fp64": np.full(4, TOL64), "fp16dev": np.full(4, 5e-2)}.get(
        precision, np.array([2e-4, 2e-4, 1e-2, 1e-3]))
    assert np.all(e <= tol), e


@pytest.mark.parametrize("precision,shape", [("fp32", (60, 110, 110)), ("fp32dev", (60, 110, 110)),
                                             ("fp32sr", (60, 110, 110)), ("fp16dev", (60, 90, 90)),
                                             ("fp16dev", (200, 71, 70))])
def test_force_strips_apart_where_other_strips_are_general(precision, shape):
    """Lattices of one strip a row, all of whose strips take the general path, and a wide one in
    binary16, where the strips with force terms keep a launch of their own (a lattice of 60 x 40
    x 40, which joins them, is the other side): two steps of a random state against the oracle,
    with the tolerances of the test above."""
    for nx, ny, nz in (shape, (60, 40, 40)):
        mask = d3.sphere_mask(nx, ny, nz, 0.4 * nx, ny / 2, nz / 2, 6.3)
        c = (int(0.4 * nx), ny // 2, nz // 2)
        box = tuple(v for m in c for v in (m - 10, m + 11))
        S0 = d3.near_rest_state3(nx, ny, nz, seed=8, amp=0.02, dtype=np.float32)
        sims = [_sim3(mask, 0.56, 0.04, precision=precision, box=box, max_record=4) for _ in range(2)]
        for g, schemes in zip(sims, (None, ())):
            g.set_populations(S0)
            g.step(2, **({} if schemes is None else {"schemes": schemes}))
        np.testing.assert_array_equal(sims[0].populations(), sims[1].populations())
        o = D.OracleSim3(mask, tau=0.56, uin=np.full((nz, ny), 0.04), box=box)
        o.set_state(S0)
        o.step(2)
        e = _force_err(sims[0].forces(), o.forces())
        print(precision, (nx, ny, nz), "force errors", e, flush=True)
        tol = np.full(4, 5e-2) if precision == "fp16dev" else np.array([2e-4, 2e-4, 1e-2, 1e-3])
        assert np.all(e <= tol), e
