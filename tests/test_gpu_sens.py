"""The sensitivity kernel at the edges of its split: one to eight rows of
cells (a wave each), tiles with a remainder, and a mesh of more than 256 tiles
(two rows to a wave), for every order, with lam = u and lam != u.

Tolerance (written here): 1e-12 of the largest value against the oracle's
dense K_s on the same vectors, a few thousand FP64 roundings."""

import numpy as np
import pytest
import torch

from oracle import bilinear_sensitivity, oracle_solve
from paper_1811_09821_amd import problems as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nelx,nely,p,d", [
    (9, 7, 1, 1), (9, 7, 1, 8), (13, 5, 2, 2), (9, 7, 2, 7), (9, 7, 3, 4), (8, 8, 3, 1), (9, 7, 4, 2), (13, 10, 4, 5),
    (5, 3, 4, 8), (130, 128, 1, 3)])
def test_sensitivity_split(cuda, nelx, nely, p, d):
    from paper_1811_09821_amd import mto

    loads = [(nelx, nely, 0.0, -1.0, 0), (nelx, 0, 0.7, 0.4, 1)]
    pr = P.uniform_random(nelx, nely, p, d, seed=40 + p, loads=loads, n_load_cases=2)
    o = oracle_solve(**pr.oracle_args())
    plan = mto.Plan(pr)
    rho = torch.tensor(pr.rho, device=cuda)
    u = torch.tensor(o["u"].ravel(), device=cuda)
    lam = torch.tensor(o["u"][::-1].copy().ravel(), device=cuda)
    for gpu, other in ((plan.sensitivity(rho, u), 0), (plan.adjoint_sensitivity(rho, u, lam), 1)):
        g = gpu.cpu().numpy().reshape(2, pr.n_cells)
        for lc in range(2):
            ref = bilinear_sensitivity(pr.nelx, pr.nely, pr.p, pr.d, pr.rho, o["u"][lc], o["u"][(lc + other) % 2])
            assert np.abs(g[lc] - ref).max() <= 1e-12 * np.abs(ref).max()
