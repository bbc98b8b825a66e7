"""PDFs at the edges of where their counters are kept: in LDS up to 8192
counters whatever the cells, up to 40000 from 12 cells per counter on (or, in a
batch, with a cell per counter in one patch), else in memory, with grids of
fewer cells than workgroups; counts exactly the oracle's."""
import numpy as np
import pytest

from gpu_util import say, torch
from oracle import diagnostics as od
from paper_1510_05061_amd import hydro

pytestmark = pytest.mark.gpu

GAMMA = 5.0 / 3.0


def state(shape, seed):
    rng = np.random.default_rng(seed)
    U = np.empty((5,) + shape)
    U[0] = rng.uniform(0.5, 2.0, shape)
    U[1:4] = rng.normal(size=(3,) + shape) * 0.1
    U[4] = rng.uniform(2.0, 3.0, shape)
    return U


@pytest.mark.parametrize("prec", [hydro.FP64, hydro.FP32])
@pytest.mark.parametrize("shape,nbins", [
    ((1, 1, 5), 8191), ((1, 1, 5), 40000), ((1, 1, 1), 1 << 20),          # in memory
    ((1, 31, 33), 8190),                                                  # 256 threads
    ((12, 8193, 1), 8191), ((12, 8192, 1), 8191),                         # 12 cells per counter
    ((80, 80, 75), 39998), ((80, 75, 79), 39998), ((80, 80, 75), 39999)])
def test_grid(prec, shape, nbins):
    say(f"pdf grid {shape} nbins={nbins} prec={prec}")
    dt = np.float64 if prec == hydro.FP64 else np.float32
    U = state(shape, 4).astype(dt).astype(np.float64)
    g = hydro.Grid(torch().from_numpy(U.astype(dt)).to("cuda:0"), 0.1, GAMMA,
                   flags=hydro.FLAG_NO_TUNE)
    for q, lo, hi in ((od.RHO, 0.6, 1.9), (od.SPEED, 0.0, 0.25)):
        got = g.pdf(q, lo, hi, nbins).cpu().numpy()
        np.testing.assert_array_equal(got, od.pdf(U, GAMMA, q, lo, hi, nbins))
    g.close()


@pytest.mark.parametrize("shapes,nbins", [
    ([(1, 1, 3)] * 3, 9000),                                   # in memory
    ([(16, 16, 16)] * 24, 8190), ([(16, 16, 16)] * 24, 8191),  # 11.99 cells per counter
    ([(16, 16, 16)] * 25, 8191),
    ([(4, 4, 4), (91, 90, 1), (2, 3, 5)], 8188),               # a cell per counter of a patch
    ([(4, 4, 4), (2, 4096, 1), (2, 3, 5)], 8191), ([(4, 4, 4), (2, 4097, 1), (2, 3, 5)], 8192),
    ([(16, 16, 16), (64, 64, 96), (1, 1, 1), (64, 48, 64)], 8192),  # several workgroups a patch
    ([(80, 80, 76), (8, 8, 8), (160, 80, 76)], 39998)])
def test_batch(shapes, nbins):
    say(f"pdf batch {len(shapes)} nbins={nbins}")
    Us = [state(s, 5 + k) for k, s in enumerate(shapes)]
    patches, off = [], 0
    for U in Us:
        nz, ny, nx = U.shape[1:]
        patches.append((off, nx, ny, nz, 0, .1, .1, .1))
        off += -(-U.size // 2) * 2
    pool = np.zeros(off)
    for U, p in zip(Us, patches):
        pool[p[0]:p[0] + U.size] = U.ravel()
    b = hydro.Batch(torch().from_numpy(pool).to("cuda:0"), patches, GAMMA,
                    flags=hydro.FLAG_NO_TUNE)
    got = b.pdf(od.RHO, 0.6, 1.9, nbins).cpu().numpy()
    np.testing.assert_array_equal(got, od.pdf(Us, GAMMA, od.RHO, 0.6, 1.9, nbins))
    b.close()
