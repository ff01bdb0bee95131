"""The density indicator at the ends of the number range: infinite, huge and
NaN densities, which the call takes as they are.

The oracle divides each term by the number of cells.  Tolerance (written
here): the same infinity or NaN, and 1e-15 of the largest term of the element
for a finite sum, as for the indicator's other tests."""

import numpy as np
import pytest
import torch

from oracle.adapt import density_indicator
from paper_1811_09821_amd import problems as P

pytestmark = pytest.mark.gpu

INF = float("inf")


@pytest.mark.parametrize("d", range(1, 9))
@pytest.mark.parametrize("values", [(INF,), (-INF,), (INF, -INF), (float("nan"),), (1.7e308,), (-1.7e308,),
                                    (5e-324,), (INF, 0.25), (-INF, float("nan"), 0.75)])
def test_density_indicator_range(cuda, d, values):
    """One element holds the values in its first cells, every second element
    none of them."""
    from paper_1811_09821_amd import mto

    pr = P.uniform_random(4, 2, 1, d, seed=90 + d)
    rho = pr.rho.copy().reshape(8, d * d)
    for e in range(0, 8, 2):
        k = min(len(values), d * d)
        rho[e, :k] = values[:k]
    g = mto.Plan(pr).density_indicator(torch.tensor(rho.ravel(), device=cuda), 1).cpu().numpy()
    with np.errstate(over="ignore"):
        ref = density_indicator(pr.d, rho.ravel(), 1)
    scale = np.nanmax(np.where(np.isfinite(rho), np.abs(rho), 1.0), axis=1) + 1.0
    for e in range(8):
        if np.isfinite(ref[e]):
            assert abs(g[e] - ref[e]) <= 1e-15 * scale[e], (e, g[e], ref[e])
        else:
            assert g[e] == ref[e] or (np.isnan(g[e]) and np.isnan(ref[e])), (e, g[e], ref[e])
