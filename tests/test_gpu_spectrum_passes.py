"""The spectra where the x-lines of a pass change: line counts around whole
passes, odd counts (the last line's partner is zeros), passes cut short so that
small grids keep enough of them, every form of an FFT stage (first or later,
steps a multiple of 16 or not), and FP32 cells over the whole range of the
type, whose velocity is formed from one reciprocal."""
import numpy as np
import pytest

from gpu_util import say, torch
from oracle import diagnostics as od
from paper_1510_05061_amd import hydro

pytestmark = pytest.mark.gpu

# (nz, ny, nx)
SHAPES = [(1, 1, 256), (1, 1025, 16), (3, 683, 32), (1, 5201, 256), (5, 1031, 96), (2, 1537, 144),
          (1, 1030, 768), (1, 1023, 1024), (1, 3001, 2), (7, 733, 27), (1, 2050, 864)]


def grid_of(U):
    dev = torch().from_numpy(U).to("cuda:0")
    return hydro.Grid(dev, (0.1,) * 3, 1.4, flags=hydro.FLAG_NO_TUNE)


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("shape", SHAPES)
def test_line_counts(shape, dtype):
    say(f"spectrum passes {shape} {dtype.__name__}")
    rng = np.random.default_rng(sum(shape))
    U = rng.standard_normal((5,) + shape).astype(dtype)
    U[0] = 0.5 + rng.random(shape, dtype=np.float32)
    g = grid_of(U)
    got, want = g.spectrum().cpu().numpy(), od.spectrum_x(U)
    # both transform in FP64, errors of a few eps log2 n of a line's norm
    np.testing.assert_allclose(got, want, rtol=1e-9, atol=1e-12 * want.sum())
    g.close()


@pytest.mark.parametrize("shape", [(1, 1024, 96), (3, 512, 864), (2, 576, 144), (27, 64, 48)])
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_shell_line_counts(shape, dtype):
    say(f"shell passes {shape} {dtype.__name__}")
    rng = np.random.default_rng(sum(shape) + 1)
    U = rng.standard_normal((5,) + shape).astype(dtype)
    U[0] = 0.5 + rng.random(shape, dtype=np.float32)
    g = grid_of(U)
    got, want = g.spectrum3d().cpu().numpy(), od.spectrum_shell(U)
    assert np.abs(got - want).max() <= 1e-12 * want.sum()
    g.close()


@pytest.mark.parametrize("scale_r,scale_m", [(1e-38, 1e-38), (1e-44, 1e-40), (3e38, 3e38),
                                             (1e30, 1e-30), (1e-20, 1e15)])
def test_fp32_range(scale_r, scale_m):
    # quotients correctly rounded to within an ulp of FP64
    say(f"spectrum of extreme FP32 cells {scale_r} {scale_m}")
    rng = np.random.default_rng(5)
    shape = (2, 3, 48)
    U = np.empty((5,) + shape, np.float32)
    U[0] = (scale_r * (0.5 + 0.5 * rng.random(shape))).astype(np.float32)
    U[1:4] = (scale_m * (2 * rng.random((3,) + shape) - 1)).astype(np.float32)
    U[4] = 1
    assert U[0].min() > 0 and np.isfinite(U).all()
    g = grid_of(U)
    want = od.spectrum_x(U)
    np.testing.assert_allclose(g.spectrum().cpu().numpy(), want, rtol=1e-9,
                               atol=1e-12 * want.sum())
    g.close()
