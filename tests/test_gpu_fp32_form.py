"""FP32 instances at tau = 1 without a body force are held as their moments
(relative to the plane references); the population form stays for every other
one and for snapshots that hold populations. Both against the FP64 oracle and
against each other."""
import numpy as np
import pytest

from helpers import oracle_solver, rel_l2

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2110_13055_amd")
from paper_2110_13055_amd import _lib as L  # noqa: E402
from paper_2110_13055_amd import Batch, Geometry, Params, Solver  # noqa: E402

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
