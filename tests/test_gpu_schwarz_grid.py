"""The bounded grid of the Schwarz application: each wave looks at 64 of its
tiles at once and takes those with a running system.  MTO_ASM_GRID caps the
blocks of a launch, which makes small plans take it: the results have to be
the same bits whichever wave takes a tile.
"""

import ctypes

import numpy as np
import pytest
import torch

from paper_1811_09821_amd import problems as P


def mto():
    from paper_1811_09821_amd import mto as m

    return m


def blocks(n_tiles):
    f = mto().lib()._ZN3mto16asm_apply_blocksEi  # mto::asm_apply_blocks(int)
    f.argtypes, f.restype = [ctypes.c_int], ctypes.c_int
    return f(n_tiles)


def test_blocks_of_a_launch(monkeypatch):
    """A block per four tiles, at most 4096 blocks, never more than the cap; what
    is not a positive number caps nothing."""
    monkeypatch.delenv("MTO_ASM_GRID", raising=False)
    assert [blocks(n) for n in (1, 4, 5, 16380, 16384, 16385, 10**6)] == [1, 1, 2, 4095, 4096, 4096, 4096]
    for cap in ("0", "-3", "x", ""):
        monkeypatch.setenv("MTO_ASM_GRID", cap)
        assert [blocks(n) for n in (5, 16385)] == [2, 4096]
    monkeypatch.setenv("MTO_ASM_GRID", "5")
    assert [blocks(n) for n in (1, 16, 20, 21, 16381)] == [1, 4, 5, 5, 5]


def problems():
    """A p = 4 design of six loads (576 tiles, two passes of up to four systems;
    the last load is absent, so its system stops at once) and one of all
    orders with three loads."""
    rng = np.random.default_rng(83)
    loads = [(48, 4 * k, 0.0, -1.0, k) for k in range(5)]
    return [P.uniform_random(48, 24, 4, 5, seed=81, loads=loads, n_load_cases=6),
            P.uniform_random(20, 12, rng.choice([1, 2, 3, 4], 240), rng.integers(1, 4, 240), 82, lo=0.1,
                             loads=[(20, 6 * k, 0.0, -1.0, k) for k in range(3)], n_load_cases=3)]


@pytest.mark.gpu
@pytest.mark.parametrize("precision", [1e-11, 1e-13])
def test_capped_grids(cuda, monkeypatch, precision):
    """Plans made, and their iterations captured, under caps of 1 (a wave
    walks several windows of 64 tiles), 2, 5 and 9 blocks against no cap."""
    prs = problems()
    rho = torch.tensor(np.concatenate([p.rho for p in prs]), device=cuda)
    monkeypatch.delenv("MTO_ASM_GRID", raising=False)
    u0, c0, g0, st0 = mto().Plan(prs, rtol=precision).solve(rho)
    assert len(set(st0["iterations"])) > 2 and min(st0["iterations"]) == 0, st0["iterations"]
    for cap in ("1", "2", "5", "9"):
        monkeypatch.setenv("MTO_ASM_GRID", cap)
        plan = mto().Plan(prs, rtol=precision)
        u, c, g, st = plan.solve(rho)
        assert torch.equal(u, u0) and torch.equal(c, c0) and torch.equal(g, g0), cap
        assert st["iterations"] == st0["iterations"], cap
        u, c, g = plan.capture(rho)
        st = plan.replay()
        assert torch.equal(u, u0) and torch.equal(c, c0) and torch.equal(g, g0), cap
        assert st["iterations"] == st0["iterations"], cap
