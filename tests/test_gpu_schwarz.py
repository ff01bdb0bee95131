"""The Schwarz application at the edges of its tiles and launches (tiles of
16, 7, 4 and 2 elements for p = 1..4, one wave each, up to four systems per
pass; a bounded grid from 4096 blocks on).

The application is checked through the solves it preconditions, against the
oracle at the tolerances of the other solve tests (u and c 1e-8, dc/drho
1e-7), and where the mesh is too large for the oracle through the true
residual, which the solve evaluates by other kernels.
"""

import numpy as np
import pytest
import torch

from oracle import oracle_solve
from paper_1811_09821_amd import problems as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p,nelx,nely", [(1, 17, 1), (1, 8, 4), (2, 7, 1), (2, 8, 3), (3, 5, 1), (3, 4, 2), (4, 3, 1),
                                         (4, 2, 3)])
@pytest.mark.parametrize("n_loads", [1, 4, 5])
def test_partial_tiles(cuda, p, nelx, nely, n_loads):
    """Last tiles full and ragged; one, four and five load cases (one, one and
    two passes), one of them without a load so that it stops at once."""
    from paper_1811_09821_amd import mto

    loads = [(nelx, k % (nely + 1), 0.3 * k, -1.0, k) for k in range(n_loads - (n_loads > 1))]
    pr = P.uniform_random(nelx, nely, p, 2, seed=60 + p, loads=loads, n_load_cases=n_loads)
    plan = mto.Plan(pr)
    u, c, g, st = plan.solve(torch.tensor(pr.rho, device=cuda))
    o = oracle_solve(**pr.oracle_args())
    assert np.linalg.norm(u.cpu().numpy() - o["u"].ravel()) < 1e-8 * np.linalg.norm(o["u"])
    assert np.all(np.abs(c.cpu().numpy() - o["c"]) <= 1e-8 * np.abs(o["c"]))
    assert np.linalg.norm(g.cpu().numpy() - o["g"].ravel()) < 1e-7 * np.linalg.norm(o["g"])


def test_bounded_grid(cuda):
    """4226 blocks of tiles: the bounded grid, each wave walking several tiles.
    A wrong or missing tile would leave its elements unsmoothed (z = 0 there)."""
    from paper_1811_09821_amd import mto

    pr = P.uniform_random(520, 520, 1, 1, seed=3, lo=0.4)
    u, c, g, st = mto.Plan(pr).solve(torch.tensor(pr.rho, device=cuda))
    assert st["status"] == 0 and st["true_rel_residual"][0] <= 1e-11
    assert st["max_iterations"] < 60, st["iterations"]


def test_residual_pass(cuda):
    """1.1 million DOFs: the residual of the second application in a pass of
    its own (below 2^20 DOFs the gather forms it)."""
    from paper_1811_09821_amd import mto

    pr = P.uniform_random(740, 740, 1, 1, seed=4, lo=0.4)
    u, c, g, st = mto.Plan(pr).solve(torch.tensor(pr.rho, device=cuda))
    assert st["status"] == 0 and st["true_rel_residual"][0] <= 1e-11
    assert st["max_iterations"] < 60, st["iterations"]
