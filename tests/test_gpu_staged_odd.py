"""Odd AA steps through the LDS stage against the same steps without it
(set_tuning's stage_odd): FP32 and FP16 populations, flow alone and fused,
body force and open x ends, with boundary voxels whose interior neighbour is
solid (they write past the stage). Both forms evaluate the same expressions on
the same inputs; the bar leaves a rounding per step and value: 12 steps of
2^-23, relative to the largest value (FP16: of its own 2^-11 in units of the
population deviations, some 1e-2 of the velocity)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2110_13055_amd")
from paper_2110_13055_amd import _lib as L  # noqa: E402
from paper_2110_13055_amd import Geometry, Params, Solver  # noqa: E402


def run(stage, dim, precision, forced, fused):
    nx, ny, nz = (45, 38, 1) if dim == 2 else (25, 22, 19)
    rng = np.random.default_rng(7)
    lab = (rng.random((nz, ny, nx)) < 0.2).astype(np.uint8)
    lab[..., :2] = lab[..., -2:] = 0
    lab[:, 3:9, 1] = 1    # end voxels without a fluid interior neighbour
    lab[:, 5:7, -2] = 1
    g = Geometry(dim=dim, nx=nx, ny=ny, nz=nz, kind=L.USER_LABELS, user_labels=lab)
    kw = dict(drive=L.BODY_FORCE, body_force=(1e-5, 4e-6, 0.0), u_in=0.0) if forced else dict(u_in=1e-3)
    s = Solver(g, Params(tau=0.8 if precision == L.FP32 else 1.0, precision=precision, **kw))
    s.set_tuning(stage_odd=1 if stage else 2)
    if fused:
        s.np_step(13, fused=True)
    else:
        s.flow_steps(13)
    return s.velocity(), s.density(), s.concentration()


@pytest.mark.parametrize("fused", [False, True], ids=["flow", "fused"])
@pytest.mark.parametrize("forced", [False, True], ids=["open", "force"])
@pytest.mark.parametrize("dim,precision", [(2, "FP32"), (3, "FP32"), (3, "FP16"), (2, "FP16")])
def test_staged_steps_match_the_others(dim, precision, forced, fused):
    a = run(True, dim, getattr(L, precision), forced, fused)
    b = run(False, dim, getattr(L, precision), forced, fused)
    assert np.abs(a[0]).max() > 1e-6
    for x, y in zip(a, b):
        eps = 2.0 ** -23 if precision == "FP32" or x is a[2] else 2.0 ** -11 * 1e-2
        assert np.abs(x - y).max() <= 13 * eps * np.abs(y).max()
