"""Workspaces of the level step: without the region of the fine face fluxes
the step takes the register launches instead, and the three ways (fused sweeps
that write face fluxes, fused sweeps with the least workspace, separate sweeps)
give the same bits; a workspace below the least is refused; nothing past the
given bytes is written."""
import ctypes

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
CFG = "x:v={v},b=512;y:q=64,s=4;z:q=64,s=4;p:g=512,d=1,f={f};w:v={v},b=256"


def up(b):
    return (b + 255) // 256 * 256


@pytest.mark.parametrize("prec", [hydro.FP64, hydro.FP32])
@pytest.mark.parametrize("g,v,boxes", [
    (2, 1, [((2, 2, 2), (4, 4, 4)), ((6, 2, 10), (20, 8, 6)), ((34, 16, 6), (6, 14, 15))]),
    (3, 2, [((10, 8, 6), (4, 4, 4)), ((2, 24, 12), (30, 6, 9))]),
    (4, 4, [((12, 8, 8), (6, 4, 5))])])
def test_level_step_workspaces(prec, g, v, boxes):
    say(f"level workspace prec={prec} g={g} v={v}")
    dt = np.float64 if prec == hydro.FP64 else np.float32
    esz = np.dtype(dt).itemsize
    C = ic.smooth_random(SHAPE, 41, gamma=GAMMA, mach=0.3).U.reshape(-1).astype(dt)
    flat, patches, off = [], [], 0
    for i, (n, _) in enumerate(boxes):
        shp = tuple(n[2 - a] + 2 * g for a in range(3))
        F = ic.smooth_random(shp, 50 + i, gamma=GAMMA, mach=0.3).U.reshape(-1)
        flat += [F, np.zeros((-F.size) % 64)]
        patches.append((off, shp[2], shp[1], shp[0], 0) + tuple(h / 2 for h in DX))
        off += F.size + (-F.size) % 64
    F = np.concatenate(flat).astype(dt)
    maxface = max(max(n[1] * n[2], n[0] * n[2], n[0] * n[1]) // 4 for n, _ in boxes)
    nreg = len(boxes) * 30 * maxface
    least = up(C.size * esz) + up(16 * nreg) + 24 * len(boxes)
    links = hydro.make_links([(i, 0) + o for i, (_, o) in enumerate(boxes)])
    outs = {}
    for way, f, size in (("faces", 1, None), ("least", 1, least), ("short", 1, -8),
                         ("separate", 0, least)):
        tc = torch().from_numpy(C).to("cuda:0")
        tf = torch().from_numpy(F).to("cuda:0")
        coarse = hydro.Batch(tc, [(0, SHAPE[2], SHAPE[1], SHAPE[0], 0) + DX], GAMMA, grav=GRAV,
                             flags=hydro.FLAG_NO_TUNE)
        fine = hydro.Batch(tf, patches, GAMMA, bc=(hydro.OUTFLOW,) * 6, grav=GRAV,
                           flags=hydro.FLAG_NO_TUNE)
        fine.config = CFG.format(v=v, f=f)
        asked = hydro.hydro_amr_step_workspace_bytes(coarse.ctx, fine.ctx, g)
        assert (asked > least) if f else (asked == least)
        size = asked if size is None else asked + size if size < 0 else size
        ws = torch().full((asked + 4096,), 0xA5, dtype=torch().uint8, device="cuda:0")
        wp = ctypes.c_void_p(ws.data_ptr())
        step = lambda nb: hydro.lib().hydro_amr_step(coarse.ctx, fine.ctx, links, len(boxes), g,
                                                     1e-3, 0, wp, nb)
        assert step(least - 1) == hydro.HYDRO_EINVAL
        for _ in range(3):
            assert step(size) == hydro.HYDRO_OK
        outs[way] = host(tc), host(tf)
        assert bool((ws[size:] == 0xA5).all())
        assert coarse.error() == fine.error() == hydro.HYDRO_OK
        coarse.close()
        fine.close()
    for way in ("least", "short", "separate"):
        for a, b in zip(outs["faces"], outs[way]):
            np.testing.assert_array_equal(a, b)
