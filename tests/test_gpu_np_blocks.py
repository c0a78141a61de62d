"""The ion solver's block preconditioner (Chebyshev sweeps over blocks of 1024
consecutive nodes, both species side by side) at the sizes where a block can
go wrong: lattices of less than a block, of exactly one, one node more, and a
ragged last block; an isolated cell with no outflow; weak and steep fields;
with the neighbour list and (ions periodic in x, flow not) without. Against
the FP64 oracle, to the implicit tests' bar (coefficients in FP32 on both sides
of the change: 1e-4 of the largest concentration)."""
import numpy as np
import pytest

from helpers import oracle_solver

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2110_13055_amd")
from paper_2110_13055_amd import _lib as L  # noqa: E402
from paper_2110_13055_amd import Geometry, Params, Potential, Solver  # noqa: E402


def channel(n_fluid, dim):
    """n_fluid fluid voxels of a small lattice, in its first rows; one isolated
    fluid cell inside inert solid."""
    nx, ny, nz = (16, 20, 1) if dim == 2 else (16, 16, 12)
    lab = np.ones((nz, ny, nx), np.uint8)
    lab.reshape(-1)[:n_fluid - 1] = 0
    lab[-1, -3:, -5:-2] = 2
    lab[-1, -2, -4] = 0  # its in-plane neighbours are inert
    if dim == 3:
        lab[-2, -2, -4] = 2
        lab[0, -2, -4] = 2  # z wraps
    return Geometry(dim=dim, nx=nx, ny=ny, nz=nz, kind=L.USER_LABELS, user_labels=lab)


@pytest.mark.parametrize("field", ["ramp", "steep", "lookup"])
@pytest.mark.parametrize("dim,n_fluid", [(2, 60), (2, 257), (3, 200), (3, 1023), (3, 1024), (3, 1025), (3, 2300)])
def test_blocks_against_the_oracle(dim, n_fluid, field):
    g = channel(n_fluid, dim)
    p = Params(u_in=1e-3, dpsi_vt=5.0, D=(0.05, 0.076), **({"np_x_bc": L.NPX_PERIODIC} if field == "lookup" else {}))
    s, o = Solver(g, p), oracle_solver(g, p)
    s.flow_steps(50)
    o.flow_steps(50)
    o.freeze_velocity()
    if field == "steep":
        pot = Potential(psi_electrode=-10.0, x_bc=(L.PSIX_DIRICHLET, L.PSIX_NEUMANN), tol=1e-12)
        s.solve_potential(pot)
        assert o.solve_potential(pot.psi_electrode, pot.x_bc, pot.psi_x, 0.0, 1e-13)[0] == 0
    s.np_implicit(20.0, 3, tol=1e-11)
    assert o.np_implicit(20.0, 3, tol=1e-13)[0] == 0
    assert np.abs(s.concentration() - o.conc()).max() <= 1e-4 * np.abs(o.conc()).max()
