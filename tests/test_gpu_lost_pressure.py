"""States that have lost their pressure: a sound speed of NaN on both sides of
an interface picks the plain flux of one side, so the step stays finite (the
sticky error flag reports the state).  A uniform state of zero or negative
pressure keeps its bits, since every flux equals its neighbour; a block of
negative pressure in an ordinary flow leaves every value finite, and the cells
that two sweeps cannot reach as they are without the block.  Every kernel shape."""
import numpy as np
import pytest

from gpu_util import host, say, torch
from paper_1510_05061_amd import hydro

pytestmark = pytest.mark.gpu

GAMMA = 1.4
NT = hydro.FLAG_NO_TUNE
GRIDS = [(0, "x:v=1,b=128;y:q=64,s=1;z:q=64,s=1"), (0, "x:v=4,b=256;y:q=64,s=4;z:q=16,s=4"),
         (0, "x:v=2,b=64,m=1;y:q=128,s=2;z:q=64,s=8"),
         (hydro.FLAG_FUSE_XY, "p:f=1;w:v=2,b=256")]
BATCHES = ["p:f=0", "p:f=1;w:v=4,b=256", "p:f=0,z=1;u:v=2,b=256"]


def uniform(shape, u, p):
    U = np.empty((5,) + shape)
    U[0] = 1.0
    for v in range(3):
        U[1 + v] = u[v]
    U[4] = p / (GAMMA - 1.0) + 0.5 * sum(v * v for v in u)
    return U


def step(U, prec, route, steps=2):
    dt = np.float64 if prec == hydro.FP64 else np.float32
    dev = torch().from_numpy(U.astype(dt)).to("cuda:0")
    nz, ny, nx = U.shape[1:]
    if isinstance(route, str):
        g = hydro.Batch(dev.view(-1), [(0, nx, ny, nz, 0, .1, .1, .1)], GAMMA, flags=NT)
        g.config = route
    else:
        g = hydro.Grid(dev, 0.1, GAMMA, flags=NT | route[0])
        g.config = route[1]
    for _ in range(steps):
        g.step(1e-3)
    out, err = host(dev), g.error()
    g.close()
    return U.astype(dt).astype(np.float64), out, err


def routes(prec):
    return [("grid", r) for r in GRIDS] + [("batch", r) for r in BATCHES
                                           if prec == hydro.FP32 or "v=4" not in r]


@pytest.mark.parametrize("prec", [hydro.FP64, hydro.FP32])
@pytest.mark.parametrize("p", [0.0, -0.25])
@pytest.mark.parametrize("u", [(0.5, -0.25, 2.0), (0.0, 1.0, -0.5), (-3.0, 0.0, 0.0)])
def test_uniform_state_without_pressure(prec, p, u):
    for kind, r in routes(prec):
        say(f"no pressure {kind} {r} prec={prec} p={p} u={u}")
        shape = (4, 64, 64) if kind == "grid" else (8, 16, 32)
        before, after, err = step(uniform(shape, u, p), prec, r)
        np.testing.assert_array_equal(after, before)
        assert err == hydro.HYDRO_ENUMERIC


@pytest.mark.parametrize("prec", [hydro.FP64, hydro.FP32])
def test_block_of_negative_pressure(prec):
    for kind, r in routes(prec):
        say(f"negative block {kind} {r} prec={prec}")
        shape = (16, 64, 64) if kind == "grid" else (16, 32, 32)
        U = uniform(shape, (0.3, -0.2, 0.1), 1.0)
        U[4, 5:9, 12:17, 14:18] -= 3.0              # p = -0.2
        before, after, err = step(U, prec, r, 1)
        assert np.isfinite(after).all() and err == hydro.HYDRO_ENUMERIC
        far = np.ones(shape, bool)      # a sweep reaches two cells along its axis
        far[3:11, 10:19, 12:20] = False
        np.testing.assert_array_equal(after[:, far], before[:, far])
