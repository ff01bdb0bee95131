"""A solve is a function of its inputs: what the plan solved before does not
move the iterations at which residuals are replaced, the bits of the results
or the iteration cap.

A full chunk within which the solve is expected to end (by the rate of an
earlier solve, or because the plan's V-cycle is the exact inverse) goes in
parts, the others whole.
"""

import numpy as np
import pytest
import torch

from oracle import oracle_solve
from paper_1811_09821_amd import problems as P

pytestmark = pytest.mark.gpu

CASES = {
    # plain fields: void regions, moduli over nine decades, residual replacements
    "plain_60x30_p2d2": (lambda: P.cantilever_uniform(60, 30, 2, 2, sigma=3.0, seed=2, solid_paths=False), {}),
    "inverter_40x20_p2d4": (lambda: P.force_inverter(40, 20, p=2, d=4), dict(rtol=1e-13)),
    "inverter_16x8_p1d2": (lambda: P.force_inverter(16, 8, p=1, d=2), dict(rtol=1e-13)),
    # one grid, solved directly: one to three iterations, and a restart on the plain field
    "mbb": (P.mbb_20x10, {}),
    "plain_40x20_p1d2": (lambda: P.cantilever_uniform(40, 20, 1, 2, sigma=3.0, seed=3, solid_paths=False),
                         dict(rtol=1e-13)),
    # ends within the second chunk of its last cycle
    "plain_61x33_p1d5_restart": (lambda: P.cantilever_uniform(61, 33, 1, 5, sigma=3.0, seed=2, solid_paths=False), {}),
    "plain_61x33_p1d5": (lambda: P.cantilever_uniform(61, 33, 1, 5, sigma=3.0, seed=8, solid_paths=False), {}),
    "p1_coarsened": (lambda: P.uniform_random(61, 33, 1, 1, seed=4), {}),
}


def mto():
    from paper_1811_09821_amd import mto as m

    return m


def same(a, b):
    return all(torch.equal(x, y) for x, y in zip(a[:3], b[:3])) and a[3]["iterations"] == b[3]["iterations"]


@pytest.mark.parametrize("key", sorted(CASES))
def test_solve_after_a_warm_start(cuda, key):
    """Cold twice, warm from the result (no or few iterations), cold, replayed:
    the cold ones equal each other and a new plan's first, bit for bit."""
    make, kw = CASES[key]
    pr = make()
    rho = torch.tensor(pr.rho, device=cuda)

    def cold(plan):
        u, c, g, st = plan.solve(rho, allow_noconv=True)
        return u.clone(), c.clone(), g.clone(), st

    plan = mto().Plan(pr, **kw)
    first = cold(plan)
    assert same(cold(plan), first)
    warm = plan.solve(rho, u0=first[0], allow_noconv=True)
    assert max(warm[3]["iterations"]) <= max(first[3]["iterations"])
    assert same(cold(plan), first)
    assert same(cold(mto().Plan(pr, **kw)), first)
    u, c, g = plan.capture(rho)
    for _ in range(2):
        st = plan.replay(allow_noconv=True)
        assert same((u, c, g, st), first)
    assert same(cold(plan), first)


@pytest.mark.parametrize("key", ["mbb", "plain_60x30_p2d2"])
def test_iteration_cap_after_a_warm_start(cuda, key):
    """max_iter is counted in whole chunks of eight, whatever came before."""
    pr = CASES[key][0]()
    rho = torch.tensor(pr.rho, device=cuda)
    u = mto().Plan(pr).solve(rho)[0]
    plan = mto().Plan(pr, max_iter=8, max_restarts=0)
    its = [plan.solve(rho, u0=u0, allow_noconv=True)[3]["iterations"][0] for u0 in (None, u, None)]
    assert its[0] == its[2] <= 8 and its[1] <= 2, its


@pytest.mark.parametrize("iters_per_launch", [2, 4, 8, 16, 28])
@pytest.mark.parametrize("rtol", [1e-11, 1e-13])
def test_chunk_in_parts(cuda, iters_per_launch, rtol):
    """The first chunk in parts at several lengths (28 is not a whole number of
    parts) against the oracle (u and c to 1e-8, dc/drho to 1e-7, as for the
    other solves)."""
    pr = CASES["plain_40x20_p1d2"][0]()
    u, c, g, st = mto().Plan(pr, iters_per_launch=iters_per_launch, rtol=rtol).solve(
        torch.tensor(pr.rho, device=cuda))
    o = oracle_solve(**pr.oracle_args())
    assert np.linalg.norm(u.cpu().numpy() - o["u"].ravel()) < 1e-8 * np.linalg.norm(o["u"])
    assert np.all(np.abs(c.cpu().numpy() - o["c"]) <= 1e-8 * np.abs(o["c"]))
    assert np.linalg.norm(g.cpu().numpy() - o["g"].ravel()) < 1e-7 * np.linalg.norm(o["g"])
