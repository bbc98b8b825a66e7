"""The fine flux registers of hydro_amr_step written by the fused sweeps: with
a fine batch that fuses x and y per patch plane, the plane and z sweeps put
the fluxes through the patch faces into the workspace and one launch gathers
them, in place of register launches that recompute those fluxes before each
sweep.  Both run the same arithmetic on the same cells, so three level steps
(both sweep orders at both levels) must agree to the rounding of the flux
expressions, at the edges of the tiles: patches of one coarse cell, uneven
extents, every lane run, two to four ghost layers, both precisions, gravity."""
import numpy as np
import pytest

import hydro_ic as ic
from gpu_util import host, say, torch
from paper_1510_05061_amd import hydro

pytestmark = pytest.mark.gpu

GAMMA = 1.4
SHAPE = (24, 24, 40)                      # coarse (nz, ny, nx)
DX = (1 / 40, 1 / 24, 1 / 24)
GRAV = (0.1, -0.2, -0.5)
BASE = "x:v={v},b=512;y:q=64,s=4;z:q=64,s=4;p:g=512,d=1,"

# ghost layers, lane run, fine interior extents (nx, ny, nz) and coarse
# offsets: every stored extent (interior + 2 g) along x and y a multiple of v
CASES = [
    (2, 1, [((2, 2, 2), (4, 4, 4)), ((6, 2, 10), (20, 8, 6)), ((34, 16, 6), (6, 14, 15))]),
    (2, 4, [((28, 24, 20), (4, 4, 4)), ((4, 8, 2), (24, 6, 8))]),
    (3, 2, [((10, 8, 6), (4, 4, 4)), ((2, 24, 12), (30, 6, 9))]),
    (4, 4, [((12, 8, 6), (4, 4, 4)), ((32, 4, 26), (16, 16, 5)), ((8, 16, 2), (20, 4, 12))]),
]


def run(prec, g, boxes, cfg, reflux):
    dt = np.float64 if prec == hydro.FP64 else np.float32
    C = ic.smooth_random(SHAPE, 41, gamma=GAMMA, mach=0.3).U
    tc = torch().from_numpy(C.reshape(-1).astype(dt)).to("cuda:0")
    coarse = hydro.Batch(tc, [(0, SHAPE[2], SHAPE[1], SHAPE[0], 0) + DX], GAMMA, grav=GRAV,
                         flags=hydro.FLAG_NO_TUNE)
    flat, patches, off = [], [], 0
    for i, (n, _) in enumerate(boxes):
        shp = tuple(n[2 - a] + 2 * g for a in range(3))
        F = ic.smooth_random(shp, 50 + i, gamma=GAMMA, mach=0.3).U.reshape(-1)
        pad = (-F.size) % 64
        flat += [F, np.zeros(pad)]
        patches.append((off, shp[2], shp[1], shp[0], 0) + tuple(h / 2 for h in DX))
        off += F.size + pad
    tf = torch().from_numpy(np.concatenate(flat).astype(dt)).to("cuda:0")
    fine = hydro.Batch(tf, patches, GAMMA, bc=(hydro.OUTFLOW,) * 6, grav=GRAV,
                       flags=hydro.FLAG_NO_TUNE)
    fine.config = cfg
    lv = hydro.AmrLevels(coarse, fine, [(i, 0) + o for i, (_, o) in enumerate(boxes)], g)
    step = 0.5 * lv.cfl_dt()
    for _ in range(3):
        lv.step(step, reflux=reflux)
    out = host(tc).astype(np.float64), host(tf).astype(np.float64)
    assert coarse.error() == fine.error() == hydro.HYDRO_OK
    coarse.close()
    fine.close()
    return out


@pytest.mark.parametrize("prec", [hydro.FP64, hydro.FP32])
@pytest.mark.parametrize("g,v,boxes", CASES)
def test_face_fluxes_equal_the_register_launches(prec, g, v, boxes):
    say(f"amr faces prec={prec} g={g} v={v}")
    cs, fs = run(prec, g, boxes, BASE.format(v=v) + "f=0", True)
    cf, ff = run(prec, g, boxes, BASE.format(v=v) + f"f=1;w:v={v},b=256", True)
    plain, _ = run(prec, g, boxes, BASE.format(v=v) + "f=0", False)
    # a register holds dt/dx F with F rounded to the state's type; the two
    # paths may contract its products differently, a few ulp of the largest
    # state value a step, carried through three steps
    eps = np.finfo(np.float64 if prec == hydro.FP64 else np.float32).eps
    ec = np.abs(cf - cs).max() / np.abs(cs).max()
    ef = np.abs(ff - fs).max() / np.abs(fs).max()
    say(f"  coarse {ec / eps:.1f} eps, fine {ef / eps:.1f} eps")
    assert max(ec, ef) <= 64 * eps
    if prec == hydro.FP64:  # the corrections themselves are far above it
        assert np.abs(plain - cs).max() / np.abs(cs).max() > 1e4 * eps
