"""Ghost prolongation of fine patches that store no ghosts: it writes nothing,
alone and in a call (and a workgroup) mixed with patches that have them; bit
for bit against the oracle, with what no patch stores left alone."""
import numpy as np
import pytest

from gpu_util import say, torch
from oracle import amr
from paper_1510_05061_amd import hydro

pytestmark = pytest.mark.gpu

BC = (hydro.PERIODIC,) * 6


def stored(pool, p):
    """Writeable (5, z, y, x) view of what patch p stores, ghosts included."""
    nx, ny, nz, ng = p[1:5]
    shape = (5, nz + 2 * ng, ny + 2 * ng, nx + 2 * ng)
    return pool[p[0]:p[0] + int(np.prod(shape))].reshape(shape)


# coarse ghost layers, ghost layers of the fine patches (one link each)
@pytest.mark.parametrize("prec", [hydro.FP64, hydro.FP32])
@pytest.mark.parametrize("ghosts_only", [False, True])
@pytest.mark.parametrize("cng,fine", [(2, [0]), (2, [0, 2, 0]), (3, [3, 0, 2, 1, 0, 4, 0, 0, 2]),
                                      (2, [0] * 130 + [2])])
def test_prolong_into_ghostless_patches(prec, ghosts_only, cng, fine):
    say(f"prolong ghostless prec={prec} ghosts_only={ghosts_only} fine={fine[:10]}")
    dt = np.float64 if prec == hydro.FP64 else np.float32
    rng = np.random.default_rng(11)
    patches, off = [], 0
    for n, ng in [((8, 8, 8), cng)] + [((8, 6, 4), g) for g in fine]:
        patches.append((off,) + n + (ng,) + tuple(1.0 / m for m in n))
        off = -(-(off + 5 * int(np.prod([m + 2 * ng for m in n]))) // 16) * 16 + 16
    pool = np.full(off, np.nan)
    for p in patches:
        S = stored(pool, p)
        S[...] = rng.uniform(0.5, 2.0, S.shape)
    pool = pool.astype(dt)
    links = [(i + 1, 0, 2, 2, 2) for i in range(len(fine))]
    dev = torch().from_numpy(pool).to("cuda:0")
    b = hydro.Batch(dev, patches, 1.4, bc=BC, flags=hydro.FLAG_NO_TUNE)
    b.prolong(links, ghosts_only=ghosts_only)
    got, want = dev.double().cpu().numpy(), pool.astype(np.float64)
    for f, c, ox, oy, oz in links:
        F = stored(want, patches[f])
        F[...] = amr.prolong(stored(want, patches[c]), cng, F, patches[f][4], (ox, oy, oz),
                             ghosts_only=ghosts_only).astype(dt)
    np.testing.assert_array_equal(got, want)     # NaN between the patches too
    b.close()
