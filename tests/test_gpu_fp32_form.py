"""The forms a state is held in, and the kernels each takes: FP32 instances at
tau = 1 without a body force as moments (relative to the plane references), FP32
populations elsewhere and for snapshots that hold populations; neighbours
through the lattice's rows, with inert solids, ragged bricks and a wrap; ion
drifts inside and beyond the flux series' range. Against the FP64 oracle and
against each other."""
import numpy as np
import pytest

from helpers import oracle_solver, rel_l2

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2110_13055_amd")
from paper_2110_13055_amd import _lib as L  # noqa: E402
from paper_2110_13055_amd import Batch, Geometry, Params, Potential, Solver  # noqa: E402

RSTATE = 16 + 7 * 4  # byte offset of the state bits in a snapshot's header


def case(**pk):
    g = Geometry(dim=3, nx=40, ny=32, nz=28, kind=L.SPHERES, porosity=0.5, r_min=3.0, r_max=6.0, seed=7)
    return g, Params(u_in=5e-4, dpsi_vt=20.0, **pk)


def as_populations(s):
    """The solver's snapshot of the rest state, marked as holding populations
    (at rest both forms are all zeros): as one written before the moment form."""
    blob = bytearray(s.snapshot())
    assert blob[RSTATE] & 8
    blob[RSTATE] &= ~8 & 0xFF
    return bytes(blob)


@pytest.mark.parametrize("streaming", [L.STREAM_AA, L.STREAM_PULL], ids=["aa", "pull"])
def test_population_snapshot_is_stepped_on_as_populations(streaming):
    g, p = case(streaming=streaming)
    a, b = Solver(g, p), Solver(g, p)
    b.restore(as_populations(b))
    for s in (a, b):
        s.flow_to_steady(tol=0.0, max_steps=44, check_every=10)  # renews the references
        s.np_step(21, fused=True)
    assert not b.snapshot()[RSTATE] & 8 and a.snapshot()[RSTATE] & 8
    # both round FP32 values of the same state: 65 steps of 6e-8 each, well below 1e-5
    assert rel_l2(a.velocity(), b.velocity()) <= 1e-5
    assert np.abs(a.concentration() - b.concentration()).max() <= 1e-5
    # the two forms in one batch, each bitwise as stepped alone
    c, d = Solver(g, p), Solver(g, p)
    c.restore(a.snapshot())
    d.restore(b.snapshot())
    bt = Batch([c, d])
    bt.advance(7, [L.MODE_FUSED, L.MODE_FUSED])
    bt.close()
    for s in (a, b):
        s.np_step(7, fused=True)
    for s, t in ((a, c), (b, d)):
        assert np.array_equal(s.velocity(), t.velocity()) and np.array_equal(s.concentration(), t.concentration())


@pytest.mark.parametrize("npx", [L.NPX_INLET_OUTLET, L.NPX_PERIODIC], ids=["open", "periodic"])
def test_fused_ions_after_renewed_references(npx):
    # the ions' mass flux is formed from moments relative to the planes' references
    # (across the periodic seam: the other end's plane)
    g, p = case(np_x_bc=npx)
    s, o = Solver(g, p), oracle_solver(g, p)
    s.flow_to_steady(tol=0.0, max_steps=303, check_every=50)
    o.flow_steps(303)
    s.np_step(61, fused=True)
    assert o.np_steps(61, fused=True) == 0
    assert rel_l2(s.velocity(), o.velocity()) <= 1e-5
    assert np.abs(s.density() - o.density()).max() <= 1e-6
    assert np.abs(s.concentration() - o.conc()).max() <= 1e-4
    s.np_step(11)  # frozen: the flux of the moments
    assert o.np_steps(11) == 0
    assert np.abs(s.concentration() - o.conc()).max() <= 1e-4


def test_snapshot_with_the_species_in_planes():
    # a snapshot written when the two species were two planes (bit 4 clear)
    g, p = case()
    s = Solver(g, p)
    s.np_step(7)
    want = s.concentration()
    blob = bytearray(s.snapshot())
    P_ = (s.n_fluid + 255) // 256 * 256
    at = 72 + (19 * 4 + 2 * 3 * 4 + 4 * 4) * P_  # behind the populations, the flux pair and the previous velocity
    for _ in range(2):
        pairs = np.frombuffer(blob, np.float32, 2 * P_, at).reshape(P_, 2)
        blob[at:at + 8 * P_] = np.ascontiguousarray(pairs.T).tobytes()
        at += 8 * P_
    blob[RSTATE] &= ~16 & 0xFF
    t = Solver(g, p)
    t.restore(bytes(blob))
    assert np.array_equal(t.concentration(), want)
    s.np_step(3)
    t.np_step(3)
    assert np.array_equal(t.concentration(), s.concentration())


@pytest.mark.parametrize("streaming", [L.STREAM_AA, L.STREAM_PULL], ids=["aa", "pull"])
@pytest.mark.parametrize("precision", [L.FP32, L.FP16, L.FP16_DEV], ids=["fp32", "fp16", "fp16dev"])
def test_population_batches_equal_members_alone(precision, streaming):
    # tau = 0.8: the batched kernels of the population forms
    specs = []
    for n, seed in ((24, 3), (33, 4)):
        g = Geometry(dim=3, nx=n, ny=n - 5, nz=n - 3, kind=L.SPHERES, porosity=0.6, r_min=3.0, r_max=5.0, seed=seed)
        specs.append((g, Params(u_in=1e-3, dpsi_vt=10.0, tau=0.8, precision=precision, streaming=streaming)))
    alone, both = [Solver(*sp) for sp in specs], [Solver(*sp) for sp in specs]
    b = Batch(both)
    for n, mode in ((9, L.MODE_FLOW), (8, L.MODE_FUSED), (5, L.MODE_IONS)):
        b.advance(n, mode)
        for s in alone:
            s.flow_steps(n) if mode == L.MODE_FLOW else s.np_step(n, fused=mode == L.MODE_FUSED)
    b.close()
    for s, t in zip(alone, both):
        assert np.array_equal(s.velocity(), t.velocity()) and np.array_equal(s.concentration(), t.concentration())
        assert np.array_equal(s.adsorbed_total(), t.adsorbed_total())


def labels(nz, ny, nx, seed, inert):
    """Random solid voxels (0.35 of them), a share of which is inert; x ends open."""
    r = np.random.default_rng(seed)
    lab = (r.random((nz, ny, nx)) < 0.35).astype(np.uint8)
    lab[(lab == 1) & (r.random(lab.shape) < inert)] = 2
    lab[:, :, :2] = lab[:, :, -2:] = 0
    return lab


@pytest.mark.parametrize("nbr_list", [0, 1])
@pytest.mark.parametrize("shape", [(17, 15, 18), (16, 33, 47), (1, 20, 33), (5, 3, 16)])
@pytest.mark.parametrize("drive", [L.INLET_OUTLET, L.BODY_FORCE], ids=["inout", "force"])
def test_rows_on_ragged_lattices_with_inert_solids(shape, drive, nbr_list):
    nz, ny, nx = shape
    g = Geometry(dim=2 if nz == 1 else 3, nx=nx, ny=ny, nz=nz, kind=L.USER_LABELS, user_labels=labels(*shape, 5, 0.4))
    pk = dict(drive=drive, body_force=(1e-5, 0.0, 0.0), u_in=0.0, Ka=2e-3) if drive == L.BODY_FORCE else dict(u_in=1e-3)
    for npx in (L.NPX_INLET_OUTLET, L.NPX_PERIODIC, L.NPX_CLOSED):
        p = Params(dpsi_vt=4.0, np_x_bc=npx, **pk)
        s, o = Solver(g, p), oracle_solver(g, p)
        s.set_tuning(nbr_list=nbr_list)
        s.flow_steps(21)
        o.flow_steps(21)
        for fused in (True, False):
            s.np_step(12, fused=fused)
            assert o.np_steps(12, fused=fused) == 0
        assert rel_l2(s.velocity(), o.velocity()) <= 1e-5
        assert np.abs(s.concentration() - o.conc()).max() <= 1e-5
        a, ao = s.adsorbed_total(), o.adsorbed_total()
        assert np.all(np.abs(a - ao) <= 1e-5 * np.abs(ao))


@pytest.mark.parametrize("fused", [False, True])
@pytest.mark.parametrize("dpsi", [0.5, 0.74, 0.9, 3.0])
def test_ion_drift_in_and_beyond_the_series_range(dpsi, fused):
    # the ramp per cell (|Pe| of the x faces): in the series' range, near its
    # end with a flow that takes some faces beyond it, and steep
    n = 24
    g = Geometry(dim=3, nx=n, ny=20, nz=18, kind=L.SPHERES, porosity=0.6, r_min=3.0, r_max=5.0, seed=2)
    p = Params(u_in=0.02, dpsi_vt=dpsi * n, D=(0.04, 0.05))
    s, o = Solver(g, p), oracle_solver(g, p)
    s.flow_steps(60)
    o.flow_steps(60)
    s.np_step(25, fused=fused)
    assert o.np_steps(25, fused=fused) == 0
    assert np.abs(s.concentration() - o.conc()).max() <= 1e-5
    m = s.mass_balance()  # solute + adsorbed + out - in is kept (FP32 fluxes, 25 steps)
    m0 = s.n_fluid * p.c0
    assert np.all(np.abs(m[:, 0] + m[:, 1] + m[:, 3] - m[:, 2] - m0) <= 1e-6 * m0)


def internal_x(lab):
    """x of the fluid nodes in the library's order (bricks of 16^3, x fastest)."""
    z, y, x = np.nonzero(lab == 0)
    nbx, nby = -(-lab.shape[2] // 16), -(-lab.shape[1] // 16)
    brick = ((z >> 4) * nby + (y >> 4)) * nbx + (x >> 4)
    return x[np.argsort((brick << 12) | ((z & 15) << 8) | ((y & 15) << 4) | (x & 15))]


def test_both_sides_of_a_face_see_the_same_density():
    # moments relative to references that jump by more than a factor of two and in
    # sign from plane to plane, where reference + (neighbour's - own) rounds: the
    # state of a flow, written relative to random references. Closed ions without
    # adsorption: the solute is kept to the rounding of each cell's flux sum, five
    # additions of values near 0.02, 1.2e-9 per cell and step, here (the flow is
    # steady) the same in all steps; four times the sum over the cells
    nz, ny, nx = 28, 32, 40
    lab = np.zeros((nz, ny, nx), np.uint8)
    lab[10:14, 8:20, 14:20] = 1
    g = Geometry(dim=3, nx=nx, ny=ny, nz=nz, kind=L.USER_LABELS, user_labels=lab)
    s = Solver(g, Params(u_in=0.02, np_x_bc=L.NPX_CLOSED, no_adsorption=1))
    s.flow_to_steady(tol=0.0, max_steps=400, check_every=100)
    s.np_step(5, fused=True)  # (applies the pending references)
    s.set_concentration(np.ones((2, s.n_fluid), np.float32))
    blob = bytearray(s.snapshot())
    head = np.frombuffer(blob, np.int32, 8, 16)  # parity, mcur, ..., rstate
    mcur, rcur = int(head[1]), int(head[7]) & 1
    assert head[7] & 8 and not head[7] & 2
    P_ = (s.n_fluid + 255) // 256 * 256
    ref = np.frombuffer(blob, np.float32, nx, 72 + 176 * P_ + 256 * rcur)
    m = np.frombuffer(blob, np.float32, 4 * P_, 72 + 16 * P_ * mcur).reshape(P_, 4)
    assert 0 < np.abs(ref).max() < 0.1
    x = internal_x(lab)
    new = np.random.default_rng(8).uniform(-0.4, 0.4, nx).astype(np.float32)
    m[:x.size, 0] += (ref - new)[x]
    ref[:] = new
    u, rho = s.velocity(), s.density()
    s.restore(bytes(blob))
    assert rel_l2(s.velocity(), u) <= 1e-5 and np.abs(s.density() - rho).max() <= 1e-6
    steps = 20
    m0 = s.mass_balance()[:, 0]
    s.np_step(steps, fused=True)
    drift = np.abs(s.mass_balance()[:, 0] - m0)
    print(f"solute drift {drift} of {s.n_fluid}")
    assert drift.max() <= 4 * 1.2e-9 * steps * np.sqrt(s.n_fluid)


@pytest.mark.parametrize("dim", [2, 3])
@pytest.mark.parametrize("form", [dict(), dict(precision=L.FP16), dict(tau=0.8), dict(tau=0.8, precision=L.FP16_DEV),
                                  dict(precision=L.MOMENTS)], ids=["fp32", "fp16", "tau0.8", "fp16dev", "moments"])
def test_drift_kernels_give_the_same_values(form, dim):
    # cell Peclet numbers of up to about 8. One call keeps the kernel that its
    # first check chooses (the fluid is at rest there), a call per step chooses anew
    # as the flow sets in, a batch for itself
    n = 40
    g = (Geometry(dim=3, nx=n, ny=24, nz=20, kind=L.SPHERES, porosity=0.6, r_min=3.0, r_max=5.0, seed=2) if dim == 3 else
         Geometry(dim=2, nx=2 * n, ny=48, nz=1, kind=L.DISKS, porosity=0.7, r_min=4.0, r_max=6.0, min_gap=2.0, seed=2,
                  walls_y=1))
    a, b, c = (Solver(g, Params(u_in=0.02, dpsi_vt=0.2 * n, D=(0.006, 0.009), **form)) for _ in range(3))
    a.np_step(60, fused=True)
    for _ in range(60):
        b.np_step(1, fused=True)
    bt = Batch([c])
    for k in (1, 19, 40):
        bt.advance(k, L.MODE_FUSED)
    assert np.abs(a.np_velocity()).max() > 4 * 0.006
    for k in range(2):
        for s in (b, c):
            assert np.array_equal(a.concentration(), s.concentration()) and np.array_equal(a.velocity(), s.velocity())
            assert np.array_equal(a.mass_balance(), s.mass_balance())
        for s in (a, b):
            s.np_step(7)
        bt.advance(7, L.MODE_IONS)
    bt.close()


@pytest.mark.parametrize("alone_in_ramp", [False, True])
def test_members_of_every_flux_form_in_one_batch(alone_in_ramp):
    # ramp, steep ramp, drift-dominated flow and a solved potential: together they
    # take the batched kernels with every form, ramps alone those without
    pk = [dict(dpsi_vt=5.0), dict(dpsi_vt=3.0)] if alone_in_ramp else \
        [dict(dpsi_vt=5.0), dict(dpsi_vt=60.0), dict(u_in=0.02, D=(0.006, 0.009)), dict()]
    alone, both = [], []
    for to in (alone, both):
        for k, q in enumerate(pk):
            g = Geometry(dim=3, nx=24 + 3 * k, ny=21, nz=20, kind=L.SPHERES, porosity=0.6, r_min=3.0, r_max=5.0, seed=k + 1)
            s = Solver(g, Params(**{"u_in": 1e-3, **q}))
            s.flow_steps(30)
            if not q:
                s.solve_potential(Potential(psi_electrode=-2.0, x_bc=(L.PSIX_DIRICHLET, L.PSIX_NEUMANN), tol=1e-8))
            to.append(s)
    b = Batch(both)
    for n, mode in ((6, L.MODE_FUSED), (5, L.MODE_IONS), (4, L.MODE_FLOW), (7, L.MODE_FUSED)):
        b.advance(n, mode)
        for s in alone:
            s.flow_steps(n) if mode == L.MODE_FLOW else s.np_step(n, fused=mode == L.MODE_FUSED)
    b.close()
    for s, t in zip(alone, both):
        assert np.array_equal(s.concentration(), t.concentration()) and np.array_equal(s.velocity(), t.velocity())
        assert np.array_equal(s.mass_balance(), t.mass_balance())
