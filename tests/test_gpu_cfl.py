"""The standalone CFL reduction at the edges of its split: grids and batches
whose cells end inside a workgroup's first trip, on it and past it (1024
cells), batches whose small patches need fewer workgroups than the largest,
and the fastest cell at the very end of a patch.  dt against its definition
in numpy, to the parity bound of dt (1e-14 relative, FP64)."""
import numpy as np
import pytest

from gpu_util import say, torch
from paper_1510_05061_amd import hydro

pytestmark = pytest.mark.gpu

GAMMA, CFL = 1.4, 0.8


def state(shape, seed):
    rng = np.random.default_rng(seed)
    U = np.empty((5,) + shape)
    U[0] = rng.uniform(0.5, 2.0, shape)
    U[1:4] = rng.normal(size=(3,) + shape) * 0.3
    U[4] = 4.0
    U[:, -1, -1, -1] = (1.0, 0.5, -9.0, 0.25, 60.0)  # the fastest cell, last in memory
    return U


def rate(U, dx):
    p = (GAMMA - 1.0) * (U[4] - 0.5 * (U[1:4] ** 2).sum(0) / U[0])
    c = np.sqrt(GAMMA * p / U[0])
    n = U.shape[:0:-1]
    return max(float(((np.abs(U[1 + a] / U[0]) + c) / dx[a]).max()) for a in range(3) if n[a] > 1)


@pytest.mark.parametrize("shape", [(1, 1, 2), (1, 33, 31), (1, 32, 32), (1, 25, 41),
                                   (5, 7, 61), (64, 64, 65), (129, 128, 127)])
def test_grid_dt(shape):
    say(f"cfl grid {shape}")
    U = state(shape, 1)
    dx = (0.1, 0.2, 0.05)
    g = hydro.Grid(torch().from_numpy(U).to("cuda:0"), dx, GAMMA, CFL, flags=hydro.FLAG_NO_TUNE)
    want = CFL / rate(U, dx)
    assert abs(g.cfl_dt() - want) <= 1e-14 * want
    g.close()


@pytest.mark.parametrize("own", [False, True])
@pytest.mark.parametrize("shapes", [[(4, 4, 4), (48, 40, 44), (2, 8, 64)], [(96, 97, 98)],
                                    [(8, 8, 8)] * 1500])
def test_batch_dt(shapes, own):
    say(f"cfl batch {len(shapes)} own={own}")
    Us = [state(s, k) for k, s in enumerate(shapes)]
    patches, off = [], 0
    for U in Us:
        nz, ny, nx = U.shape[1:]
        patches.append((off, nx, ny, nz, 0, 1.0 / nx, 1.0 / ny, 1.0 / nz))
        off += -(-U.size // 2) * 2
    pool = np.zeros(off)
    for U, p in zip(Us, patches):
        pool[p[0]:p[0] + U.size] = U.ravel()
    b = hydro.Batch(torch().from_numpy(pool).to("cuda:0"), patches, GAMMA, CFL,
                    flags=hydro.FLAG_NO_TUNE | (hydro.BATCH_PER_PATCH_DT if own else 0))
    want = np.array([CFL / rate(U, p[5:8]) for U, p in zip(Us, patches)])
    assert abs(b.cfl_dt() - want.min()) <= 1e-14 * want.min()
    if own:
        np.testing.assert_allclose(b.times()[1], want, rtol=1e-14, atol=0.0)
    b.close()
