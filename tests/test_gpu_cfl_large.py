"""The standalone CFL reduction on both sides of the size from which a thread
holds two cells in flight in place of four (2^24): the fastest cell anywhere
and at the very end, grids and patches; dt against its definition, to the
parity bound of dt (1e-14 relative in FP64; 1e-5 for speeds formed in FP32)."""
import numpy as np
import pytest

from gpu_util import say, torch
from paper_1510_05061_amd import hydro

pytestmark = pytest.mark.gpu

GAMMA, CFL = 1.4, 0.8


@pytest.mark.parametrize("prec", [hydro.FP64, hydro.FP32])
@pytest.mark.parametrize("batch", [False, True])
@pytest.mark.parametrize("shape", [(256, 256, 256), (255, 257, 256), (300, 241, 236)])
def test_large_dt(prec, batch, shape):
    say(f"cfl large {shape} batch={batch} prec={prec}")
    t = torch()
    cells = int(np.prod(shape))
    dt = t.float64 if prec == hydro.FP64 else t.float32
    dx = (0.1, 0.2, 0.05)
    off = 5 * 64
    pool = t.empty(off + 5 * cells, dtype=dt, device="cuda:0")
    for S in (pool[:off].view(5, -1), pool[off:].view(5, -1)):
        S[0], S[1:4], S[4] = 1.0, 0.125, 4.0
    U = pool[off:].view((5,) + shape)
    if batch:
        g = hydro.Batch(pool, [(0, 4, 4, 4, 0) + dx, (off,) + shape[::-1] + (0,) + dx], GAMMA, CFL,
                        flags=hydro.FLAG_NO_TUNE)
    else:
        g = hydro.Grid(U, dx, GAMMA, CFL, flags=hydro.FLAG_NO_TUNE)
    nz, ny, nx = shape
    for k, (z, y, x) in enumerate([(nz - 1, ny - 1, nx - 1), (0, 0, 0), (nz // 2, ny - 1, nx // 3)]):
        cell = (1.0, 0.5, -9.0, 0.25, 60.0 + k)
        keep = U[:, z, y, x].clone()
        U[:, z, y, x] = t.tensor(cell, dtype=dt, device="cuda:0")
        g.state_changed()
        r, m, e = cell[0], cell[1:4], cell[4]
        c = np.sqrt(GAMMA * (GAMMA - 1.0) * (e - 0.5 * sum(v * v for v in m) / r) / r)
        want = CFL / max((abs(v) / r + c) / h for v, h in zip(m, dx))
        assert abs(g.cfl_dt() - want) <= (1e-14 if prec == hydro.FP64 else 1e-5) * want
        U[:, z, y, x] = keep
    g.close()
