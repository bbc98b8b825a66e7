"""Workspaces of the shell spectrum: the least size (rows of nx / 2 + 1
values back to back) is taken and gives the bits of the reported size, a byte
less is refused, and nothing past the given bytes is written."""
import ctypes

import numpy as np
import pytest

import hydro_ic as ic
from gpu_util import say, torch
from oracle import diagnostics as od
from paper_1510_05061_amd import hydro

pytestmark = pytest.mark.gpu

PARTIALS = 2048                       # partial spectra kept by the binning


def least_bytes(shape, shells):
    nz, ny, nx = shape
    cells = (nx // 2 + 1) * ny * nz
    return sum((b + 255) // 256 * 256
               for b in (48 * cells, 8 * cells, 8 * PARTIALS * shells, 16 * (nx + ny + nz)))


@pytest.mark.parametrize("prec", [hydro.FP64, hydro.FP32])
@pytest.mark.parametrize("shape", [(8, 6, 2), (1, 1, 1), (9, 4, 3), (12, 16, 24), (6, 32, 96),
                                   (4, 8, 128), (3, 2, 162), (16, 8, 256), (2, 2, 1024)])
def test_least_workspace(prec, shape):
    say(f"shell spectrum workspace {shape} prec={prec}")
    U = ic.smooth_random(shape, seed=8, gamma=1.4).U
    dt = np.float64 if prec == hydro.FP64 else np.float32
    g = hydro.Grid(torch().from_numpy(U.astype(dt)).to("cuda:0"), (0.1, 0.2, 0.3), 1.4,
                   flags=hydro.FLAG_NO_TUNE)
    want = g.spectrum3d().cpu().numpy()
    ref = od.spectrum_shell(U.astype(dt).astype(np.float64))
    assert np.abs(want - ref).max() <= 1e-12 * ref.sum()
    nbytes, nb = g.spectrum3d_workspace()
    least = least_bytes(shape, nb)
    assert least <= nbytes <= 1.125 * least
    work = torch().full((nbytes + 4096,), 0xA5, dtype=torch().uint8, device="cuda:0")
    out = torch().empty(nb, dtype=torch().float64, device="cuda:0")
    wp, op = ctypes.c_void_p(work.data_ptr()), ctypes.c_void_p(out.data_ptr())
    with pytest.raises(hydro.HydroError) as e:
        hydro.hydro_diag_spectrum3d(g.ctx, wp, least - 1, op)
    assert e.value.status == hydro.HYDRO_EINVAL
    for size in sorted({least, (least + nbytes) // 2, max(least, nbytes - 1)}):
        work.fill_(0xA5)
        hydro.hydro_diag_spectrum3d(g.ctx, wp, size, op)
        np.testing.assert_array_equal(out.cpu().numpy(), want)
        assert bool((work[size:] == 0xA5).all())
    g.close()
