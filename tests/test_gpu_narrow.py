"""The sum-factorised product on tiles of 16 columns (plans of at most 256 such
tiles; 512 where no element has more than 2 x 2 cells and some have p >= 3)
and of 64: the same bits for a design, whatever else is in its plan.

Tolerance against the oracle's assembled K x: 1e-13 in the 2-norm, as derived
for the other products' tests.
"""

import numpy as np
import pytest
import torch

from oracle.solve import assemble, free_mask
from paper_1811_09821_amd import problems as P

pytestmark = pytest.mark.gpu


def mto():
    from paper_1811_09821_amd import mto as m

    return m


def vector(pr, seed):
    K, space, *_ = assemble(pr.nelx, pr.nely, pr.p, pr.d, pr.rho, pr.E0, pr.Emin, pr.q, pr.nu)
    free = free_mask(space, pr.supports)
    x = np.random.default_rng(seed).standard_normal((pr.n_load_cases, space.n_dof))
    x[:, ~free] = 0.0
    ref = (K @ x.T).T
    ref[:, ~free] = 0.0
    return x.ravel(), ref.ravel()


def filler(large):
    """4224 or 17600 elements: 264 or 1100 narrow tiles by itself, so that the
    plan takes tiles of 64 columns, 66 (each split over four waves) or 275."""
    nelx, nely = (160, 110) if large else (66, 64)
    return P.uniform_random(nelx, nely, 3, 3, seed=1, lo=0.4)


def check(pr, cuda, seed):
    """Alone and beside each filler, against the oracle and each other."""
    x, ref = vector(pr, seed)
    out = []
    for prs in ([pr], [pr, filler(False)], [pr, filler(True)]):
        plan = mto().Plan(prs)
        rho = torch.tensor(np.concatenate([q.rho for q in prs]), device=cuda)
        xs = torch.zeros(plan.info["n_u"], dtype=torch.float64, device=cuda)
        xs[:x.size] = torch.tensor(x, device=cuda)
        y = plan.apply_stiffness(rho, xs)[:x.size]
        err = np.linalg.norm(y.cpu().numpy() - ref) / np.linalg.norm(ref)
        assert err < 1e-13, (pr.name, len(prs), err)
        out.append((y, plan.sensitivity(rho, xs)[:pr.n_cells * pr.n_load_cases], plan.jacobi_diagonal(rho)))
    for other in out[1:]:
        for a, b in zip(out[0], other):
            assert torch.equal(a, b[:a.numel()])


@pytest.mark.parametrize("p,d", [(p, d) for p in (1, 2, 3, 4) for d in range(1, 9)])
def test_every_group(cuda, p, d):
    """35 columns: two full narrow tiles and a ragged one; one ragged tile of 64."""
    check(P.uniform_random(7, 5, p, d, seed=300 + 10 * p + d), cuda, d)


def test_mixed_orders_and_loads(cuda):
    rng = np.random.default_rng(6)
    p, d = rng.choice([1, 2, 3, 4], 200), rng.integers(1, 6, 200)
    loads = [(20, 3 * k, 0.0, -1.0, k) for k in range(3)]
    check(P.uniform_random(20, 10, p, d, 11, loads=loads, n_load_cases=3), cuda, 5)


@pytest.mark.parametrize("p,d,nelx,nely", [(3, 3, 64, 64), (3, 3, 241, 17), (3, 2, 128, 64), (4, 1, 241, 34)])
def test_edges_of_the_rule(cuda, p, d, nelx, nely):
    """256 and 257 narrow tiles (d > 2), 512 and 513 (d <= 2)."""
    check(P.uniform_random(nelx, nely, p, d, seed=8, lo=0.2), cuda, 6)


@pytest.mark.parametrize("p,d", [(1, 5), (2, 3), (3, 2), (4, 4)])
def test_solves(cuda, p, d):
    """Products, vertex updates and stopped systems of whole solves: the same
    bits alone and beside twelve designs of 750 elements.  (All meshes are their
    own coarsest grid: the largest one sets the number of levels for all.)"""
    loads = [(13, 0, 0.0, -1.0, 0), (13, 5, 1.0, 0.5, 1)]
    pr = P.uniform_random(13, 7, p, d, seed=21, loads=loads, n_load_cases=3)  # the third load is absent
    u, c, g, st = mto().Plan(pr).solve(torch.tensor(pr.rho, device=cuda))
    prs = [pr] + [P.uniform_random(30, 25, 1, 1, seed=30 + k, lo=0.4) for k in range(12)]
    ub, cb, gb, sb = mto().Plan(prs).solve(torch.tensor(np.concatenate([q.rho for q in prs]), device=cuda))
    assert torch.equal(ub[:u.numel()], u) and torch.equal(cb[:c.numel()], c) and torch.equal(gb[:g.numel()], g)
    assert sb["iterations"][:3] == st["iterations"]
