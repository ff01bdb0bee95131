"""The QR-error kernel at the edges of its tiles: every order with one row of
cells, four, five and eight (halves of the cell tables), and one, two, four,
five and nine load cases (single, pairs, one and more passes).

Tolerance (written here): |eps - eps_oracle| <= 1e-9 per element on the same
displacements, as in the indicator's other tests (different factorisations of
the same SPD system, refined in double-double)."""

import numpy as np
import pytest
import torch

from oracle import oracle_solve
from oracle.qr import qr_error
from paper_1811_09821_amd import problems as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p", [1, 2, 3, 4])
@pytest.mark.parametrize("d,n_loads", [(1, 1), (4, 2), (5, 4), (8, 1), (2, 5), (3, 9)])
def test_qr_edges(cuda, p, d, n_loads):
    from paper_1811_09821_amd import mto

    nelx, nely = 4, 3
    loads = [(nelx, k % (nely + 1), 0.3 * k, -1.0, k) for k in range(n_loads)]
    pr = P.uniform_random(nelx, nely, p, d, seed=90 + p, loads=loads, n_load_cases=n_loads, lo=0.3)
    u = oracle_solve(**pr.oracle_args())["u"]
    plan = mto.Plan(pr)
    eps = plan.qr_error(torch.tensor(pr.rho, device=cuda), torch.tensor(u.ravel(), device=cuda)).cpu().numpy()
    ref = qr_error(pr.nelx, pr.nely, pr.p, pr.d, pr.rho, u)
    assert np.abs(eps - np.asarray(ref).ravel()).max() <= 1e-9
