"""The tile-shape cache: a line counts only for what it was measured on, the
candidates it was chosen among and, for a whole plan, the plan's groups."""

import numpy as np
import pytest
import torch

from paper_1811_09821_amd import problems as P

pytestmark = pytest.mark.gpu


def mto():
    from paper_1811_09821_amd import mto as m

    return m


def mixed(pd, seed=46, nelx=16, nely=8):
    """All (p, d) of `pd` in equal parts."""
    pd = np.array(pd)[np.arange(nelx * nely) % len(pd)]
    return P.uniform_random(nelx, nely, pd[:, 0], pd[:, 1], seed)


def entries(path):
    return [ln.split() for ln in path.read_text().splitlines() if not ln.startswith("#")]


def write(path, lines):
    path.write_text("".join(" ".join(v) + "\n" for v in lines))


def autotune(pr, path, cuda):
    plan = mto().Plan(pr)
    return plan, plan.autotune(torch.tensor(pr.rho, device=cuda), cache=str(path))


def test_file_without_the_candidates(cuda, tmp_path):
    """A file as it was before the sum-factorised product was a candidate (seven
    fields): its dense shapes and its plan-level choice are read, not taken, and
    replaced."""
    pr = mixed([(1, 1), (2, 2), (4, 5)])
    path = tmp_path / "tiles.txt"
    plan, _ = autotune(pr, path, cuda)
    groups = plan.info["n_groups"]
    old = [v[:7] for v in entries(path)]
    for v in old:
        v[4], v[5], v[6] = ("2", "0", "0.001") if v[1] == "0" else ("1", "1", "0.001")
    write(path, old)
    _, rep = autotune(pr, path, cuda)
    assert "cached" not in rep and "all groups:" in rep, rep
    assert rep.count("(sum-factorised)") == groups, rep
    new = entries(path)
    assert len(new) == groups + 1 and all(len(v) == (9 if v[1] == "0" else 8) for v in new), new
    assert all(v[6] != "0.001" for v in new), new
    _, rep = autotune(pr, path, cuda)
    assert rep.count("cached") == groups and "all groups:" not in rep, rep


def test_plans_of_other_groups(cuda, tmp_path):
    """Two plans of three groups each and as many columns: the choice measured
    on one is not taken for the other, and each finds its own again."""
    a, b = mixed([(1, 1), (2, 2), (4, 5)]), mixed([(1, 2), (2, 1), (3, 2)])
    path = tmp_path / "tiles.txt"
    autotune(a, path, cuda)
    _, rep = autotune(b, path, cuda)
    assert "all groups:" in rep, rep
    plans = [v for v in entries(path) if v[1] == "0"]
    assert len(plans) == 2 and plans[0][:4] == plans[1][:4], plans
    for pr in (a, b):
        _, rep = autotune(pr, path, cuda)
        assert rep.count("cached") == 3 and "all groups:" not in rep, rep


@pytest.mark.parametrize("line", ["gfx950 3 4 13 1", "gfx950 3 4 13 3 1 1.0 2", "gfx950 3 4 13 1 x 1.0 2",
                                  "gfx950 5 4 13 1 1 1.0"])
def test_malformed_line(cuda, tmp_path, line):
    path = tmp_path / "tiles.txt"
    path.write_text(line + "\n")
    with pytest.raises(mto().MtoError) as ei:
        autotune(mixed([(1, 1)]), path, cuda)
    assert ei.value.code == mto().MTO_EINVAL


@pytest.mark.parametrize("config", [1, 2, 3])
def test_shipped_file(cuda, config):
    """The committed choices are those of the workload configurations' groups."""
    import os
    import shutil
    import tempfile

    prs = P.config(config)
    with tempfile.TemporaryDirectory() as d:
        path = shutil.copy(os.path.join(os.path.dirname(P.__file__), "tiles_gfx950.txt"), d)
        plan, rep = autotune(prs, path, cuda)
    assert rep.count("cached") == plan.info["n_groups"] and "all groups:" not in rep, rep
