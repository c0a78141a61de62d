"""The FP32 correction solves' block preconditioner (Chebyshev sweeps over
blocks of 1024 consecutive nodes, zero outside) at the sizes where a block can
go wrong: lattices of less than a block, of exactly one, one node more, and a
ragged last block; isolated cells (no face at all); with and without the
neighbour list. Against the FP64 oracle, to the FP32 rounding of the stored
potential (two ulps of the largest value)."""
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


@pytest.mark.parametrize("x_bc", [(L.PSIX_DIRICHLET, L.PSIX_NEUMANN), (L.PSIX_PERIODIC, L.PSIX_PERIODIC)],
                         ids=["list", "lookup"])
@pytest.mark.parametrize("dim,n_fluid", [(2, 40), (2, 257), (3, 200), (3, 1023), (3, 1024), (3, 1025), (3, 2300)])
def test_blocks_against_the_oracle(dim, n_fluid, x_bc):
    g = channel(n_fluid, dim)
    p = Params(u_in=1e-3)
    s, o = Solver(g, p), oracle_solver(g, p)
    # (no charge: the isolated cell, a row of zeros in A, could not balance it)
    pot = Potential(psi_electrode=-7.0, x_bc=x_bc, psi_x=(1.0, 0.0), kappa2=0.0, tol=1e-12)
    s.solve_potential(pot)
    assert o.solve_potential(-7.0, x_bc, (1.0, 0.0), 0.0, 1e-14)[0] == 0
    assert np.abs(s.potential() - o.potential()).max() <= 2 * 7.0 * 2.0 ** -23
