"""The reactive source where its route changes: substep counts around the
one from which the chain is stepped in scaled species, links frozen out (a
rate of zero, or one so small that the scale factor leaves its range) in some
zones and not in others, and overflowing scale factors; FP64 against the
oracle to the parity bound of the source (1e-12 relative)."""
import numpy as np
import pytest

from gpu_util import say, torch
from oracle import burn
from paper_1510_05061_amd import hydro

pytestmark = pytest.mark.gpu

GAMMA = 1.4


def network(M, kind):
    rng = np.random.default_rng(M)
    A, Ta = 10.0 ** rng.uniform(-1, 4, M - 1), rng.uniform(0.0, 3.0, M - 1)
    if kind == "frozen":      # exp(-Ta / T) from 1e-30 to 1e-320 over the zones
        Ta[(M - 1) // 2] = 90.0
    elif kind == "zero":
        A[M // 2 - 1] = 0.0
    elif kind == "stiff":     # scale factors far above their upper bound
        A[:] = 10.0 ** np.where(np.arange(M - 1) % 2 == 0, 14, 1)
    return A, Ta, rng.uniform(0.01, 0.1, M - 1)


@pytest.mark.parametrize("kind", ["plain", "frozen", "zero", "stiff"])
@pytest.mark.parametrize("nsub", [7, 8, 9, 11, 64])
@pytest.mark.parametrize("M", [2, 3, 13, 20])
def test_burn_routes(kind, nsub, M):
    say(f"burn {kind} nsub={nsub} M={M}")
    rng = np.random.default_rng(nsub)
    shape = (3, 5, 37)                       # a ragged last workgroup
    U = np.empty((5,) + shape)
    U[0] = rng.uniform(0.5, 2.0, shape)
    U[1:4] = rng.normal(size=(3,) + shape) * 0.1
    p = U[0] * 10.0 ** rng.uniform(-0.7, 0.3, shape)     # T from 0.2 to 2
    U[4] = p / (GAMMA - 1.0) + 0.5 * (U[1:4] ** 2).sum(0) / U[0]
    X = rng.uniform(0.0, 1.0, (M,) + shape)
    X /= X.sum(0)
    A, Ta, q = network(M, kind)
    dU, dX = torch().from_numpy(U).to("cuda:0"), torch().from_numpy(X).to("cuda:0")
    g = hydro.Grid(dU, 0.1, GAMMA, flags=hydro.FLAG_NO_TUNE)
    g.burn(dX, A, Ta, q, 1e-2, nsub)
    wantU, wantX = burn.burn(U, X, GAMMA, A, Ta, q, 1e-2, nsub)
    np.testing.assert_allclose(dX.cpu().numpy(), wantX, rtol=1e-12, atol=1e-300)
    np.testing.assert_allclose(dU.cpu().numpy()[4], wantU[4], rtol=1e-12)
    g.close()
