"""The Kelly indicator's patches (16 x 4 elements and their neighbours) at
their edges: meshes of one patch, of one element more, of fewer, of one row or
column, for every largest order the kernel is built for.

Tolerance (written here): 1e-10 of the largest value, as for the indicator's
other tests: the jumps are differences of two gradients, so the error scales
with the gradients."""

import numpy as np
import pytest
import torch

from oracle import oracle_solve
from oracle.adapt import kelly_indicator
from paper_1811_09821_amd import problems as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p", [1, 2, 3, 4])
@pytest.mark.parametrize("nelx,nely", [(16, 4), (17, 5), (15, 3), (33, 2), (2, 9), (5, 1)])
def test_kelly_patches(cuda, nelx, nely, p):
    from paper_1811_09821_amd import mto

    pr = P.uniform_random(nelx, nely, p, 2, seed=80 + p)
    u = oracle_solve(**pr.oracle_args())["u"]
    g = mto.Plan(pr).kelly_indicator(torch.tensor(u.ravel(), device=cuda)).cpu().numpy()
    ref = kelly_indicator(pr.nelx, pr.nely, pr.p, u).ravel()
    assert np.abs(g - ref).max() <= 1e-10 * np.abs(ref).max()
