"""Ghost fill and prolongation at the edges of their walks, bit for bit
against the oracle: odd and even ghost depths (children beyond the stored
shell), rows whose x pairs are not aligned to pairs of elements, and link
counts below, at and above the eight that share out over the XCDs."""
import numpy as np
import pytest

from gpu_util import say, torch
from oracle import amr
from paper_1510_05061_amd import hydro

pytestmark = pytest.mark.gpu

P, O, R = hydro.PERIODIC, hydro.OUTFLOW, hydro.REFLECT


def stored(pool, p):
    """Writeable (5, z, y, x) view of what patch p stores, ghosts included."""
    nx, ny, nz, ng = p[1:5]
    strides = [pool.itemsize * n for n in (p[10], p[9], p[8], 1)]
    return np.lib.stride_tricks.as_strided(
        pool[p[0]:], (5, nz + 2 * ng, ny + 2 * ng, nx + 2 * ng), strides)


def pool_of(shapes, ng, dtype, slack):
    """Patches with ng NaN ghost layers, `slack` spare elements per row."""
    rng = np.random.default_rng(7)
    patches, off = [], 0
    for nz, ny, nx in shapes:
        rp = nx + 2 * ng + slack
        sp, m = rp * (ny + 2 * ng), nz + 2 * ng
        patches.append((off, nx, ny, nz, ng, 1.0 / nx, 1.0 / nx, 1.0 / nx, rp, sp, sp * m,
                        ng * (1 + rp + sp)))
        off = -(-(off + 5 * sp * m) // 16) * 16
    pool = np.full(off, np.nan)
    for p in patches:
        stored(pool, p)[(slice(None),) + (slice(ng, -ng),) * 3] = rng.uniform(
            0.5, 2.0, (5, p[3], p[2], p[1]))
    return pool.astype(dtype), patches


@pytest.mark.parametrize("prec", [hydro.FP64, hydro.FP32])
@pytest.mark.parametrize("ng", [2, 3])
@pytest.mark.parametrize("slack", [0, 3])
@pytest.mark.parametrize("nlinks", [1, 8, 11])
def test_prolong_edges(prec, ng, slack, nlinks):
    say(f"prolong edges prec={prec} ng={ng} slack={slack} links={nlinks}")
    dt = np.float64 if prec == hydro.FP64 else np.float32
    shapes = [(9, 8, 10)] * nlinks + [(8, 6, 10)] * nlinks
    pool, patches = pool_of(shapes, ng, dt, slack)
    links = [(nlinks + i, i, 2, 2, 2) for i in range(nlinks)]
    dev = torch().from_numpy(pool).to("cuda:0")
    b = hydro.Batch(dev, patches, 1.4, bc=(P, P, O, R, R, R), flags=hydro.FLAG_NO_TUNE)
    b.fill_ghosts()
    want = pool.astype(np.float64)
    ref = [amr.fill_ghosts(stored(want, p), ng, (P, P, O, R, R, R)) for p in patches]
    b.prolong(links)
    b.prolong(links, ghosts_only=True)
    got = dev.double().cpu().numpy()
    for f, c, ox, oy, oz in links:
        F = amr.prolong(ref[c], ng, ref[f], ng, (ox, oy, oz))
        F = amr.prolong(ref[c], ng, F, ng, (ox, oy, oz), ghosts_only=True)
        np.testing.assert_array_equal(stored(got, patches[c]), ref[c])
        np.testing.assert_array_equal(stored(got, patches[f]), F.astype(dt).astype(float))
    spare = np.ones(pool.shape, bool)   # what no patch stores keeps its NaN
    for p in patches:
        stored(spare, p)[...] = False
    assert np.isnan(got[spare]).all()
    b.close()


@pytest.mark.parametrize("prec", [hydro.FP64, hydro.FP32])
@pytest.mark.parametrize("shape,ng", [((1, 1, 70), 3), ((1, 5, 3), 7), ((40, 3, 2), 1)])
def test_fill_edges(prec, shape, ng):
    say(f"fill edges prec={prec} {shape} ng={ng}")
    dt = np.float64 if prec == hydro.FP64 else np.float32
    for bc in ((P,) * 6, (R, O, P, P, O, R)):
        pool, patches = pool_of([shape, (4, 4, 4)], ng, dt, 1)
        dev = torch().from_numpy(pool).to("cuda:0")
        b = hydro.Batch(dev, patches, 1.4, bc=bc, flags=hydro.FLAG_NO_TUNE)
        b.fill_ghosts()
        got = dev.double().cpu().numpy()
        for p in patches:
            want = amr.fill_ghosts(stored(pool.astype(np.float64), p), ng, bc)
            np.testing.assert_array_equal(stored(got, p), want)
        b.close()
