"""GPU parity of the sum-factorised element product (the default product;
tile shape ks = -3) against the oracle's assembled K x.

Tolerance, from the arithmetic: every entry is a sum of at most 2 n + d
rounded products per factor, three factors deep, so its error is below
about 3 (2 n + d) eps = 60 eps of the sum of the terms' magnitudes; 1e-13 in
the 2-norm, the bound of the other products' tests, leaves a factor of 7.
"""

import numpy as np
import pytest
import torch

from oracle.solve import assemble, free_mask
from paper_1811_09821_amd import problems as P

pytestmark = pytest.mark.gpu


def check(pr, cuda, seed):
    from paper_1811_09821_amd import mto

    K, space, *_ = assemble(pr.nelx, pr.nely, pr.p, pr.d, pr.rho, pr.E0, pr.Emin, pr.q, pr.nu)
    free = free_mask(space, pr.supports)
    x = np.random.default_rng(seed).standard_normal((pr.n_load_cases, space.n_dof))
    x[:, ~free] = 0.0
    ref = (K @ x.T).T
    ref[:, ~free] = 0.0
    plan = mto.Plan(pr)
    plan.set_tile(1, -3)
    y = plan.apply_stiffness(torch.tensor(pr.rho, device=cuda), torch.tensor(x.ravel(), device=cuda)).cpu().numpy()
    err = np.linalg.norm(y - ref.ravel()) / np.linalg.norm(ref)
    assert err < 1e-13, (pr.name, err)


@pytest.mark.parametrize("p,d", [(p, d) for p in (1, 2, 3, 4) for d in range(1, 9)])
def test_split_tiles(cuda, p, d):
    """One ragged tile of 35 columns split over four waves, by chains of cell
    rows (d = 3, 4, 6..8) or chains and components (d = 1, 2, 5)."""
    check(P.uniform_random(7, 5, p, d, seed=200 + 10 * p + d), cuda, d)


@pytest.mark.parametrize("p,d,nelx,nely", [(1, 2, 132, 125), (2, 5, 150, 110), (2, 6, 150, 110), (4, 2, 130, 127)])
def test_many_tiles(cuda, p, d, nelx, nely):
    """Just over 256 tiles: orders 1 and 2 go one tile to a wave (a partial
    last block and a ragged last tile), p = 2, d = 6 and p = 4 are split by
    chains."""
    check(P.uniform_random(nelx, nely, p, d, seed=7, lo=0.3), cuda, 3)


def test_mixed_tiles(cuda):
    """Split and whole tiles of all orders in one launch, two load cases,
    neighbouring waves of a block holding tiles of different orders."""
    rng = np.random.default_rng(5)
    p = rng.choice([1, 2, 3, 4], size=150 * 60, p=[0.45, 0.45, 0.05, 0.05])
    d = rng.integers(1, 5, 150 * 60)
    check(P.uniform_random(150, 60, p, d, 9, loads=[(150, 20, 0.0, -1.0, 0), (150, 3, 1.0, 0.0, 1)], n_load_cases=2),
          cuda, 4)
