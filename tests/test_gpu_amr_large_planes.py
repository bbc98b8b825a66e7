"""Ghost prolongation of an odd number of layers on patches whose planes end
just below 4 GiB (the limit of the kernels' 32-bit offsets), by their pitches:
every stored ghost cell bit for bit against the oracle, the interior and the
cells around the patch left alone."""
import numpy as np
import pytest

from gpu_util import say, torch
from oracle import amr
from paper_1510_05061_amd import hydro

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,n,ng", [(hydro.FP32, (2, 2, 2), 1), (hydro.FP64, (4, 2, 2), 1),
                                       (hydro.FP32, (4, 2, 6), 3)])
def test_odd_shell_of_a_plane_of_4_gib(prec, n, ng):
    t = torch()
    dt, esz = (np.float64, 8) if prec == hydro.FP64 else (np.float32, 4)
    # (plane + slab pitch) elements just fit 2^32 bytes
    m = [k + 2 * ng for k in n]
    sz = ((1 << 32) // esz - 1) // (m[2] + 1)
    sy = sz // m[1]
    plane = sz * m[2]
    say(f"odd shell prec={prec} n={n} ng={ng} plane={plane * esz} bytes")
    cn, cg = (10, 9, 11), 3
    csize = 5 * int(np.prod([k + 2 * cg for k in cn]))
    off = -(-csize // 64) * 64 + 64
    rng = np.random.default_rng(3)
    C = rng.uniform(0.5, 2.0, (5,) + tuple(k + 2 * cg for k in cn[::-1])).astype(dt)
    pool = t.full((off + 5 * plane + 64,), 7.0, dtype=getattr(t, np.dtype(dt).name),
                  device="cuda:0")
    pool[:csize] = t.from_numpy(C.reshape(-1)).to("cuda:0")
    patches = [(0,) + cn + (cg, .1, .1, .1),
               (off,) + n + (ng, .05, .05, .05, sy, sz, plane, ng * (1 + sy + sz))]
    b = hydro.Batch(pool, patches, 1.4, flags=hydro.FLAG_NO_TUNE)
    b.prolong([(1, 0, 3, 4, 3)], ghosts_only=True)
    v, k, j, i = np.meshgrid(np.arange(5), *(np.arange(q) for q in m[::-1]), indexing="ij")
    idx = off + v.astype(np.int64) * plane + k * sz + j * sy + i
    got = pool[t.from_numpy(idx.reshape(-1)).to("cuda:0")].cpu().numpy().reshape(idx.shape)
    want = amr.prolong(C, cg, np.full(idx.shape, 7.0), ng, (3, 4, 3), ghosts_only=True).astype(dt)
    np.testing.assert_array_equal(got, want)
    # nothing else was written: as many cells differ from 7 as the shell holds
    assert int((pool[off - 64:] != 7.0).sum()) == int((want != 7.0).sum())
    np.testing.assert_array_equal(pool[:csize].cpu().numpy(), C.reshape(-1))
    b.close()
    del pool
    t.cuda.empty_cache()
