"""Large read-backs (16 MiB and more, which several host threads move through a
pinned area) from a solver on hipStreamPerThread, a handle that names another
stream in every thread: they wait for the steps queued by the caller; and while
another thread captures a graph: the area is made and freed without a trace in
the capture."""
import threading

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


@pytest.mark.parametrize("own", [False, True], ids=["per_thread", "own"])
def test_reads_wait_for_the_streams_steps(own):
    torch = pytest.importorskip("torch")
    s, t = solver(torch.cuda.Stream() if own else PerThread()), solver()
    for n in (150, 151):
        s.flow_steps(n)  # still running when the copy is asked for
        u = s.velocity()
        assert u.nbytes >= 16 << 20
        t.flow_steps(n)
        assert np.array_equal(u, t.velocity())
    assert s.snapshot() == s.snapshot()


def test_another_threads_capture_goes_on():
    import torch
    s = solver()
    s.flow_steps(3)
    torch.cuda.synchronize()
    x = torch.zeros(64, device="cuda")
    g, st, seen = torch.cuda.CUDAGraph(), torch.cuda.Stream(), []

    def read_and_close():
        seen.append(s.velocity())  # makes the area
        s.close()                  # the last solver: frees it

    with torch.cuda.stream(st):
        x.add_(0)
        st.synchronize()
        g.capture_begin()  # mode "global": unsafe calls of any thread would end it
        x.add_(1)
        t = threading.Thread(target=read_and_close)
        t.start()
        t.join()
        x.add_(1)
        g.capture_end()
    for k in range(3):
        g.replay()
        torch.cuda.synchronize()
        assert torch.all(x == 2 * (k + 1))
    r = solver()
    r.flow_steps(3)
    assert np.array_equal(seen[0], r.velocity())
