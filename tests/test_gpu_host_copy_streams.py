"""Large read-backs (16 MiB and more, which several host threads move) from a
solver on hipStreamPerThread, a handle that names another stream in every
thread: they wait for the steps queued by the caller."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2110_13055_amd")
from paper_2110_13055_amd import Geometry, Params, Solver  # noqa: E402


class PerThread:
    """hipStreamPerThread where a torch stream is expected."""
    cuda_stream = 2

    def synchronize(self):
        import torch
        torch.cuda.synchronize()


def solver(stream=None):
    return Solver(Geometry(dim=3, nx=136, ny=128, nz=128, kind=P.SPHERES, porosity=0.9, r_min=3.0, r_max=6.0, seed=3),
                  Params(u_in=1e-3), stream=stream)


def test_per_thread_stream():
    s, t = solver(PerThread()), solver()
    for n in (150, 151):
        s.flow_steps(n)  # still running when the copy is asked for
        u = s.velocity()
        assert u.nbytes >= 16 << 20
        t.flow_steps(n)
        assert np.array_equal(u, t.velocity())
    assert s.snapshot() == s.snapshot()
