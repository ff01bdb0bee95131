"""mto_set_tile refuses what the plan cannot run."""

import pytest

from paper_1811_09821_amd import problems as P

pytestmark = pytest.mark.gpu


def test_sum_factorised_product_needs_the_mfma_path(cuda):
    from paper_1811_09821_amd import mto

    plan = mto.Plan(P.uniform_random(4, 3, 2, 2, seed=1), kernel_path=mto.PATH_PLAIN)
    for p, d in ((0, 0), (2, 2)):
        with pytest.raises(mto.MtoError) as ei:
            plan.set_tile(1, -3, p=p, d=d)
        assert ei.value.code == mto.MTO_EINVAL
    plan = mto.Plan(P.uniform_random(4, 3, 2, 2, seed=1))
    plan.set_tile(1, -3, p=2, d=2)
    with pytest.raises(mto.MtoError) as ei:
        plan.set_tile(1, -3, p=3, d=2)
    assert ei.value.code == mto.MTO_EINVAL
