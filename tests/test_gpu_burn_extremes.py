"""The reactive source where Ta / T leaves the range of FP64 or T is no
ordinary number: links switched off by a huge Ta, temperatures so small that
Ta / T overflows or 1 / T does, infinite, zero, negative and undefined ones,
Ta of zero among them; FP64 against the oracle to the parity bound of the
source (1e-12 relative), with NaN and infinities where the oracle has them,
and ordinary zones beside them as if they were alone."""
import numpy as np
import pytest

from gpu_util import say, torch
from oracle import burn
from paper_1510_05061_amd import hydro

pytestmark = pytest.mark.gpu

GAMMA = 2.0                     # p = E - m^2 / (2 rho): T is set without rounding
TEMPS = [1.0, 0.5, 1e-300, 3e-305, 1e-308, 4e-309, 1e-310, 5e-324, 0.0, -0.0, 1e300, 1.5e308,
         np.inf, -0.7, -1e-300, -3e-309, np.nan, 2.0]


@pytest.mark.parametrize("nsub", [3, 16])      # the plain and the scaled route
@pytest.mark.parametrize("Ta", [[1e308, 0.3, 0.0], [0.0, 1e308, 1.7e308], [0.2, 0.4, 1e10],
                                [1e-305, 3e-310, 0.5], [-0.5, 0.0, 1e-3], [700.0, 745.0, 1.0]])
def test_burn_at_extreme_temperatures(nsub, Ta):
    say(f"burn extremes nsub={nsub} Ta={Ta}")
    T = np.array(TEMPS + [1.0] * (64 - len(TEMPS) % 64)).reshape(1, 1, -1)
    U = np.zeros((5,) + T.shape)
    U[0] = 1.0
    U[4] = T                                    # p = E, T = p / 1
    rng = np.random.default_rng(5)
    X = rng.uniform(0.1, 1.0, (4,) + T.shape)
    X /= X.sum(0)
    A, q = np.array([2.0, 30.0, 0.5]), np.zeros(3)
    dU, dX = torch().from_numpy(U).to("cuda:0"), torch().from_numpy(X).to("cuda:0")
    g = hydro.Grid(dU, 0.1, GAMMA, flags=hydro.FLAG_NO_TUNE)
    g.burn(dX, A, Ta, q, 1e-2, nsub)
    with np.errstate(all="ignore"):
        want = burn.burn(U, X, GAMMA, A, np.array(Ta), q, 1e-2, nsub)[1]
    np.testing.assert_allclose(dX.cpu().numpy(), want, rtol=1e-12, atol=1e-300)
    g.close()


@pytest.mark.parametrize("nsub", [3, 16])
@pytest.mark.parametrize("hk", [1e300, 4.4e307, 4.6e307, 1e308, 1.7e308])
def test_burn_at_the_stiffest_links(nsub, hk):
    """h k up to the top of the range, where 1 / (1 + h k) is subnormal (a
    spacing of 2^-1074 against 5e-309: relative 2^-50)."""
    say(f"burn stiffest nsub={nsub} hk={hk}")
    U = np.zeros((5, 1, 1, 64))
    U[0] = U[4] = 1.0
    X = np.random.default_rng(6).uniform(0.05, 0.25, (4, 1, 1, 64))
    A, Ta, q = np.array([hk, 2.0, hk]), np.zeros(3), np.zeros(3)
    dU, dX = torch().from_numpy(U).to("cuda:0"), torch().from_numpy(X).to("cuda:0")
    g = hydro.Grid(dU, 0.1, GAMMA, flags=hydro.FLAG_NO_TUNE)
    g.burn(dX, A, Ta, q, float(nsub), nsub)       # h = 1
    with np.errstate(all="ignore"):
        want = burn.burn(U, X, GAMMA, A, Ta, q, float(nsub), nsub)[1]
    np.testing.assert_allclose(dX.cpu().numpy(), want, rtol=1e-12, atol=1e-300)
    g.close()
