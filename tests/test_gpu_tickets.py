"""Work items of the persistent batch sweeps: each taken once, whatever the
number of workgroups (one, a few, as many as there are items, many more) and
however they are handed out (tickets drawn an item ahead, or round robin).
The items are independent and the totals have one partial each, so states and
FP64 totals must be the same bits in every case, for every kernel that takes
items (packed lane runs, x march, column march, patch planes, x-z planes),
one dt or a dt per patch, over both sweep orders."""
import numpy as np
import pytest

import hydro_ic as ic
from gpu_util import host, say, torch
from paper_1510_05061_amd import hydro

pytestmark = pytest.mark.gpu

GAMMA = 1.4
SMALL = [(16, 16, 16), (48, 32, 16), (32, 16, 24), (16, 24, 8)]      # (nx, ny, nz)
LONG = [(144, 4, 6), (136, 10, 4)]
COLS = "y:q=64,s=2;z:q=64,s=2;"
KERNELS = {
    "separate": (SMALL, "x:v=4,b=128;" + COLS + "p:g={g},d={d},f=0"),
    "march": (LONG, "x:v=2,b=128,m=1;" + COLS + "p:g={g},d={d},f=0"),
    "plane": (SMALL, "x:v=4,b=128;" + COLS + "p:g={g},d={d},f=1;w:v=2,b=256"),
    "zplane": (SMALL, "x:v=4,b=128;" + COLS + "p:g={g},d={d},f=1,z=1;w:v=2,b=256;u:v=2,b=256"),
}


def run(prec, sizes, own, cfg):
    dt = np.float64 if prec == hydro.FP64 else np.float32
    flat, patches, off = [], [], 0
    for i, (nx, ny, nz) in enumerate(sizes):
        U = ic.smooth_random((nz, ny, nx), 60 + i, gamma=GAMMA, mach=0.4).U.reshape(-1)
        pad = (-U.size) % 64
        flat += [U, np.zeros(pad)]
        patches.append((off, nx, ny, nz, 0, 1 / nx, 1 / ny, 1 / nz))
        off += U.size + pad
    dev = torch().from_numpy(np.concatenate(flat).astype(dt)).to("cuda:0")
    flags = hydro.FLAG_NO_TUNE | (hydro.BATCH_PER_PATCH_DT if own else 0)
    b = hydro.Batch(dev, patches, GAMMA, grav=(0.0, -0.1, 0.2), flags=flags)
    b.config = cfg
    for _ in range(4):
        b.step()
    out, tot, t = host(dev), list(b.totals()), b.times()
    assert b.error() == hydro.HYDRO_OK
    b.close()
    return out, tot, t


@pytest.mark.parametrize("own", [False, True])
@pytest.mark.parametrize("prec", [hydro.FP64, hydro.FP32])
@pytest.mark.parametrize("kernel", KERNELS)
def test_every_item_once(kernel, prec, own):
    sizes, cfg = KERNELS[kernel]
    say(f"items {kernel} prec={prec} own={own}")
    ref = run(prec, sizes, own, cfg.format(g=7, d=0))
    for g, d in [(1, 0), (1, 1), (7, 1), (24, 1), (96, 1), (4096, 0), (4096, 1)]:
        out, tot, t = run(prec, sizes, own, cfg.format(g=g, d=d))
        np.testing.assert_array_equal(out, ref[0], err_msg=f"g={g} d={d}")
        assert tot == ref[1] and t == ref[2], (g, d)
