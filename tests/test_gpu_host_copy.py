"""Large read-backs (16 MiB and more) go through a pinned staging area in
pieces: every byte arrives, from one thread or from several at once (one has
the area, the others the runtime's copy), and after the area was given back."""
import threading

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2110_13055_amd")
from paper_2110_13055_amd import Geometry, Params, Solver  # noqa: E402


def solver(n=104, seed=3):
    s = Solver(Geometry(dim=3, nx=n, ny=n, nz=n + 3, kind=P.SPHERES, porosity=0.7, r_min=3.0, r_max=6.0, seed=seed),
               Params(u_in=1e-3, dpsi_vt=10.0))
    s.flow_steps(7)
    s.np_step(5, fused=True)
    return s


def test_large_reads_are_whole_from_several_threads():
    for _ in range(2):  # the second time on an area made again
        s = solver()
        r = np.random.default_rng(1).random((2, s.n_fluid), dtype=np.float32)
        s.set_concentration(r)
        assert np.array_equal(s.concentration(), r)
        blobs = {}
        others = [solver(seed=5), solver(seed=6)]
        want = [o.snapshot() for o in others]
        blob = s.snapshot()
        assert len(blob) > 60 << 20  # more pieces than the area has

        def read(k, o):
            blobs[k] = [o.snapshot() for _ in range(4)]

        th = [threading.Thread(target=read, args=(k, o)) for k, o in enumerate(others)]
        for t in th:
            t.start()
        for t in th:
            t.join()
        for k in range(2):
            assert all(b == want[k] for b in blobs[k])
        u = solver()
        u.restore(blob)
        assert np.array_equal(u.concentration(), r) and np.array_equal(u.velocity(), s.velocity())
        del s, u, others
