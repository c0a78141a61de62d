"""An FP16 instance of more than 2^29 fluid nodes: a node's concentrations lie
beyond a 32-bit byte offset there, so that its ion steps have kernels of their
own. Fluid at rest in an open box, random concentrations, fused steps of both
parities, an ion-only step and the same from a batch: plain diffusion,
C' = C + D sum(C_N - C), here in FP64 on the layers that hold the last nodes and
on the first ones, which 32-bit offsets would have mixed. One step rounds the
FP32 flux sum (below 3) and the update's remainder: 1e-6 is twice three steps'."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2110_13055_amd")
from paper_2110_13055_amd import _lib as L  # noqa: E402
from paper_2110_13055_amd import Batch, Geometry, Params, Solver  # noqa: E402

NX, NY, NZ = 832, 832, 784
D = (0.05, 0.076)
LAYERS = 8  # compared on either side of the seam z = 0


def start(rows):
    """Concentrations of one species on lexicographic x-y layers, from the node number."""
    n = (np.asarray(rows, np.uint64)[:, None] * np.uint64(NX * NY) + np.arange(NX * NY, dtype=np.uint64)).astype(np.uint32)
    n *= np.uint32(2654435761)
    n >>= np.uint32(8)
    return 0.5 + n.astype(np.float32) / np.float32(1 << 24)


def diffuse(c, d):
    """One step on layers (z, y, x), y periodic, x closed; the outer layers lose their neighbours."""
    out = -6.0 * c
    out += np.roll(c, 1, 1) + np.roll(c, -1, 1)
    out[:, :, 1:] += c[:, :, :-1]
    out[:, :, :-1] += c[:, :, 1:]
    out[:, :, 0] += c[:, :, 0]
    out[:, :, -1] += c[:, :, -1]
    out[1:] += c[:-1]
    out[:-1] += c[1:]
    return c + d * out


def check(s, want):
    got = s.concentration().reshape(2, NZ, NY, NX)
    for sp in range(2):
        at = np.concatenate([got[sp, NZ - LAYERS:], got[sp, :LAYERS]])
        inner = slice(3, 2 * LAYERS - 3)
        err = np.abs(at[inner] - want[sp][inner]).max()
        assert err <= 1e-6, f"species {sp}: {err}"


def test_ion_steps_beyond_two_to_the_29_nodes():
    torch = pytest.importorskip("torch")
    assert NX * NY * NZ > 2 ** 29
    if torch.cuda.mem_get_info()[0] < 160 << 30:
        pytest.skip("needs 160 GiB of free GPU memory")
    g = Geometry(dim=3, nx=NX, ny=NY, nz=NZ, kind=L.USER_LABELS, user_labels=np.zeros((NZ, NY, NX), np.uint8))
    s = Solver(g, Params(u_in=0.0, Ka=1e-3, D=D, np_x_bc=L.NPX_CLOSED, precision=L.FP16))
    c0 = np.empty((2, NZ, NX * NY), np.float32)
    for z in range(0, NZ, 16):
        c0[0, z:z + 16] = start(range(z, z + 16))
    c0[1] = c0[0][::-1]
    s.set_concentration(c0.reshape(2, -1))
    want = [np.concatenate([c0[sp, NZ - LAYERS:], c0[sp, :LAYERS]]).astype(np.float64).reshape(2 * LAYERS, NY, NX)
            for sp in range(2)]
    del c0
    print("fused, both parities, and ions alone", flush=True)
    s.np_step(2, fused=True)
    s.np_step(1)
    for sp in range(2):
        for _ in range(3):
            want[sp] = diffuse(want[sp], D[sp])
    check(s, want)
    print("batched", flush=True)
    start_c = s.concentration().reshape(2, NZ, NY, NX)
    want = [np.concatenate([start_c[sp, NZ - LAYERS:], start_c[sp, :LAYERS]]).astype(np.float64) for sp in range(2)]
    b = Batch([s])
    b.advance(1, L.MODE_IONS)
    b.advance(2, L.MODE_FUSED)
    b.close()
    for sp in range(2):
        for _ in range(3):
            want[sp] = diffuse(want[sp], D[sp])
    check(s, want)
    assert not np.any(s.velocity()[0, ::4097])
