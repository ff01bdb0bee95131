"""The density filter's two entry forms on both sides of the rule between them
(offsets of 16 bits: 511 elements of 64 cells to a row still fit, 520 do not) and
at the edges of its slices and batches.

Tolerance (written here): max-norm relative error 1e-14 for W rho and W^T g, as
in the filter's other tests (the same positive-weight terms, weights formed in
a different order)."""

import numpy as np
import pytest
import torch

from oracle import filter_matrix
from paper_1811_09821_amd import problems as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nelx,nely,d,R", [
    (509, 2, 8, 0.3), (511, 2, 8, 0.3), (520, 2, 8, 0.3), (520, 3, 8, 0.05), (1, 1, 1, 0.3), (1, 1, 8, 0.3), (8, 8, 1, 1.1),
    (13, 5, 1, 3.0), (9, 7, 3, 0.5), (65, 1, 1, 1.5)])
def test_filter_forms(cuda, nelx, nely, d, R):
    from paper_1811_09821_amd import mto

    pr = P.uniform_random(nelx, nely, 1, d, seed=3)
    F = mto.Filter(pr, R)
    rng = np.random.default_rng(nelx)
    x, gt = rng.uniform(0.0, 1.0, pr.n_cells), rng.standard_normal(pr.n_cells)
    W = filter_matrix(pr.nelx, pr.nely, pr.d, R)
    for got, ref in ((F.apply(torch.tensor(x, device=cuda)), W @ x), (F.grad(torch.tensor(gt, device=cuda)), W.T @ gt)):
        assert np.abs(got.cpu().numpy() - ref).max() <= 1e-14 * np.abs(ref).max()
