"""The reactive source on compositions far above one (number densities, to the
top of the range of FP64), where a species scaled by up to 2^400 would
overflow: against the oracle to the parity bound of the source (1e-12
relative), zones of ordinary and of huge species side by side."""
import numpy as np
import pytest

from gpu_util import say, torch
from oracle import burn
from paper_1510_05061_amd import hydro

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nsub", [7, 16])          # the plain and the scaled route
@pytest.mark.parametrize("M", [2, 13])
@pytest.mark.parametrize("top", [1e100, 1e180, 1e188, 1e250, 1e306])
def test_burn_of_large_species(nsub, M, top):
    say(f"burn large species nsub={nsub} M={M} top={top}")
    rng = np.random.default_rng(9)
    shape = (1, 2, 75)
    U = np.zeros((5,) + shape)
    U[0] = 1.0
    U[4] = rng.uniform(0.5, 2.0, shape)
    X = rng.uniform(0.05, 1.0, (M,) + shape)
    X[:, :, :, ::2] *= top
    X[M // 2, :, :, 1::10] *= top                  # one huge species in the zone
    A, Ta, q = 10.0 ** rng.uniform(-1, 3, M - 1), np.linspace(0.1, 60.0, M - 1), np.zeros(M - 1)
    dU, dX = torch().from_numpy(U).to("cuda:0"), torch().from_numpy(X).to("cuda:0")
    g = hydro.Grid(dU, 0.1, 1.4, flags=hydro.FLAG_NO_TUNE)
    g.burn(dX, A, Ta, q, 1e-2, nsub)
    want = burn.burn(U, X, 1.4, A, Ta, q, 1e-2, nsub)[1]
    assert np.isfinite(want).all()
    np.testing.assert_allclose(dX.cpu().numpy(), want, rtol=1e-12, atol=0.0)
    g.close()
