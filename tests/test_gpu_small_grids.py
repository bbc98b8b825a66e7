"""Steps that their last sweep ends (at most 2048 workgroups), and tiles of 16
and 32 columns: states bit for bit those of 64-column tiles, totals, time and
dt, at the edges of both rules; the configurations that stay refused."""
import numpy as np
import pytest

import hydro_ic as ic
from gpu_util import gpu_grid, host, say, torch
from paper_1510_05061_amd import hydro

pytestmark = pytest.mark.gpu

P_, O_, R_ = hydro.PERIODIC, hydro.OUTFLOW, hydro.REFLECT


def totals_of(U, P):
    """(FP64 totals, sums of magnitudes) of a state with phi = -(g . x)."""
    vol = float(np.prod(P.dx))
    z, y, x = np.meshgrid(*[(np.arange(n) + 0.5) * d for n, d in zip(U.shape[1:], P.dx[::-1])],
                          indexing="ij")
    phi = -(P.grav[0] * x + P.grav[1] * y + P.grav[2] * z)
    q = np.concatenate([U, (U[4] + U[0] * phi)[None]])
    return q.sum((1, 2, 3)) * vol, np.abs(q).sum((1, 2, 3)) * vol


def steps(P, prec, cfg, n=4):
    g, dev = gpu_grid(P, prec=prec, config=cfg)
    out = []
    for _ in range(n):
        g.step()
        out.append(g.totals())
    state, t = host(dev), g.time()
    g.state_changed()
    assert out[-1] == g.totals()                # the replay takes the same path
    want, scale = totals_of(state, P)
    # m cells summed in any order: within m eps of the sum of magnitudes
    assert (np.abs(np.array(out[-1]) - want) <= 2.0 ** -52 * state[0].size * scale + 1e-300).all()
    assert g.error() == hydro.HYDRO_OK
    g.close()
    return state, t


@pytest.mark.parametrize("prec", [hydro.FP64, hydro.FP32])
@pytest.mark.parametrize("q,s", [(16, 4), (16, 16), (32, 2), (32, 8), (32, 16)])
def test_narrow_tiles(prec, q, s):
    # 13 x 11 and 13 x 17 columns: ragged last tiles, segments of 1 to 9 cells
    say(f"narrow tiles q={q} s={s} prec={prec}")
    P = ic.smooth_random((17, 11, 13), seed=5, bc=(P_, P_, O_, R_, R_, O_), grav=(0.1, -0.2, 0.3))
    a, ta = steps(P, prec, f"y:q={q},s={s};z:q={q},s={s}")
    b, tb = steps(P, prec, "y:q=64,s=1;z:q=64,s=1")
    np.testing.assert_array_equal(a, b)
    assert ta == tb


@pytest.mark.parametrize("shape,cfg", [((1, 1, 2), "x:v=1,b=64"), ((1, 1, 1024), "x:v=2,b=512"),
                                       ((2, 256, 512), "z:q=64,s=1"),    # 2048 partials
                                       ((2, 257, 512), "z:q=64,s=1"),    # 2056
                                       ((2, 32, 512), "z:q=16,s=4")])    # 1024 narrow tiles
def test_step_ended_by_its_last_sweep(shape, cfg):
    say(f"step tail {shape} {cfg}")
    P = ic.smooth_random(shape, seed=6)
    a, ta = steps(P, hydro.FP64, cfg)
    b, tb = steps(P, hydro.FP64, "x:v=4,b=256" if shape[2] > 64 else None)
    np.testing.assert_array_equal(a, b)
    assert ta == tb


def test_refused_tiles():
    P = ic.smooth_random((2, 33, 512), seed=7)      # 16896 columns: 1056 tiles of 16
    g, _ = gpu_grid(P)
    for bad in ("z:q=16,s=4", "z:q=48,s=4", "z:q=32,s=1", "y:q=8,s=8"):
        with pytest.raises(hydro.HydroError):
            g.config = bad
    g.config = "z:q=32,s=4"
    g.close()
    pool = torch().ones((5, 8, 8, 8), device="cuda:0")
    pool[4] = 4.0
    b = hydro.Batch(pool.view(-1), [(0, 8, 8, 8, 0, .1, .1, .1)], 1.4, flags=hydro.FLAG_NO_TUNE)
    with pytest.raises(hydro.HydroError):
        b.config = "y:q=16,s=4"
    b.close()
