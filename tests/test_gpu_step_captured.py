"""Steps captured by the caller into a HIP graph against the same steps
launched directly, and hydro_profile_step (launches with events between)
against hydro_step: the same bits, time, dt and totals.  The graph holds an
even and an odd step, and is replayed several times with the program's own work
and synchronisations in between.  Grids that their last sweep ends, grids that a
bookkeeping launch ends, fused windows, batches with one dt and with their own."""
import numpy as np
import pytest

import hydro_ic as ic
from gpu_util import host, say, to_device, torch
from paper_1510_05061_amd import hydro

pytestmark = pytest.mark.gpu

P_, O_, R_ = hydro.PERIODIC, hydro.OUTFLOW, hydro.REFLECT
NT = hydro.FLAG_NO_TUNE


def grid(shape, cfg=None, flags=NT):
    P = ic.smooth_random(shape, seed=71, bc=(P_, P_, O_, R_, R_, O_) if shape[0] > 1 else (P_,) * 6,
                         grav=(0.1, -0.2, 0.3) if shape[0] > 1 else (0.0,) * 3)

    def make(prec, stream):
        dev = to_device(P.U, prec)
        g = hydro.Grid(dev, P.dx, P.gamma, P.cfl, P.bc, P.grav, flags=flags, stream=stream)
        if cfg:
            g.config = cfg
        return g, dev
    return make


def batch(count, flags=NT, cfg=None):
    specs = ic.batch_specs(count, seed=3, sizes=(16, 32))

    def make(prec, stream):
        dt = np.float64 if prec == hydro.FP64 else np.float32
        pool, patches = ic.batch_pool(specs, ng=4, dtype=dt, pad_rows=32)
        dev = torch().from_numpy(pool).to("cuda:0")
        b = hydro.Batch(dev, patches, 5.0 / 3.0, flags=flags, stream=stream)
        if cfg:
            b.config = cfg
        return b, dev
    return make


CASES = {
    "tube": grid((1, 1, 200)),
    "small": grid((17, 11, 13)),
    "many partials": grid((2, 257, 512), "z:q=64,s=1"),
    "fused": grid((16, 128, 128), "p:f=1;w:v=2,b=256", flags=NT | hydro.FLAG_FUSE_XY),
    "batch": batch(12),
    "batch fused, tickets": batch(12, cfg="p:g=64,d=1,f=1;w:v=2,b=256"),
    "batch own dt": batch(12, flags=NT | hydro.BATCH_PER_PATCH_DT),
}


def result(obj, dev):
    out = host(dev), obj.time()[0], obj.totals(), obj.cfl_dt()
    assert obj.error() == hydro.HYDRO_OK
    return out


def same(a, b):
    np.testing.assert_array_equal(a[0], b[0])
    assert a[1:] == b[1:]


@pytest.mark.parametrize("prec", [hydro.FP64, hydro.FP32])
@pytest.mark.parametrize("case", list(CASES))
def test_captured_steps(case, prec):
    say(f"captured {case} prec={prec}")
    t = torch()
    s = t.cuda.Stream()
    s.wait_stream(t.cuda.current_stream())
    with t.cuda.stream(s):
        a, da = CASES[case](prec, s)
        b, db = CASES[case](prec, s)
        for _ in range(2):                 # the first step forms its dt
            a.step()
            b.step()
    t.cuda.synchronize()
    graph = t.cuda.CUDAGraph()
    with t.cuda.graph(graph, stream=s):
        a.step()
        a.step()
    junk = t.zeros(1 << 16, device="cuda:0")
    for _ in range(4):
        with t.cuda.stream(s):
            graph.replay()
            b.step()
            b.step()
        t.cuda.synchronize()
        junk += 1.0
        assert float(junk.sum()) > 0.0
        same((host(da), a.time()[0], a.totals()), (host(db), b.time()[0], b.totals()))
    with t.cuda.stream(s):
        same(result(a, da), result(b, db))
    a.close()
    b.close()


@pytest.mark.parametrize("prec", [hydro.FP64, hydro.FP32])
@pytest.mark.parametrize("case", list(CASES))
def test_profiled_steps(case, prec):
    say(f"profiled {case} prec={prec}")
    a, da = CASES[case](prec, None)
    b, db = CASES[case](prec, None)
    for _ in range(4):
        a.profile_step()
        b.step()
    same(result(a, da), result(b, db))
    a.close()
    b.close()


@pytest.mark.parametrize("prec", [hydro.FP64, hydro.FP32])
@pytest.mark.parametrize("fuse", [0, 1])
def test_captured_level_steps(fuse, prec):
    say(f"captured level steps fuse={fuse} prec={prec}")
    t = torch()
    dt = np.float64 if prec == hydro.FP64 else np.float32
    C = ic.smooth_random((20, 18, 16), 41, gamma=1.4, mach=0.3).U.reshape(-1).astype(dt)
    F = ic.smooth_random((14, 12, 16), 42, gamma=1.4, mach=0.3).U.reshape(-1).astype(dt)
    dx = (1 / 16, 1 / 18, 1 / 20)

    def make(stream):
        tc, tf = (t.from_numpy(x.copy()).to("cuda:0") for x in (C, F))
        coarse = hydro.Batch(tc, [(0, 16, 18, 20, 0) + dx], 1.4, flags=NT, stream=stream)
        fine = hydro.Batch(tf, [(0, 16, 12, 14, 0) + tuple(h / 2 for h in dx)], 1.4,
                           bc=(O_,) * 6, flags=NT, stream=stream)
        fine.config = f"p:g=64,d=1,f={fuse};w:v=2,b=256"
        return hydro.AmrLevels(coarse, fine, [(0, 0, 5, 6, 7)], 4), tc, tf

    s = t.cuda.Stream()
    s.wait_stream(t.cuda.current_stream())
    with t.cuda.stream(s):
        a, ac, af = make(s)
        b, bc, bf = make(s)
        for lv in (a, b):
            lv.step(1e-3)
    t.cuda.synchronize()
    graph = t.cuda.CUDAGraph()
    with t.cuda.graph(graph, stream=s):
        a.step(1e-3)
        a.step(1e-3)
    junk = t.zeros(1 << 16, device="cuda:0")
    for _ in range(4):
        with t.cuda.stream(s):
            graph.replay()
            b.step(1e-3)
            b.step(1e-3)
        t.cuda.synchronize()
        junk += 1.0
        assert float(junk.sum()) > 0.0
        np.testing.assert_array_equal(host(ac), host(bc))
        np.testing.assert_array_equal(host(af), host(bf))
    for lv in (a, b):
        lv.coarse.close()
        lv.fine.close()
