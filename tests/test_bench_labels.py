"""What bench.py says of the element product follows what the plan launches, not
the kernels its groups would take one by one (CPU)."""

import pytest

import bench
from paper_1811_09821_amd import problems as P

CHOSEN = "p=1 d=2 ncol=1 ks=4: chosen\np=2 d=2 ncol=1 ks=-3: chosen\n"
ALL = "p=1 d=2 ncol=1 ks=-3: chosen\np=2 d=2 ncol=1 ks=-3: chosen\n"
DENSE = {(1, 2): 2 * 4 * 8**2, (2, 2): 2 * 4 * 18**2}
FACTORED = {(1, 2): 2 * 2 * (16 * 8 + (2 * 4 + 2) * 2), (2, 2): 2 * 2 * (16 * 27 + (2 * 9 + 3) * 2)}


@pytest.mark.parametrize("report,factored,kernel,bound", [
    ("product: fused (one launch for all groups)\n" + ALL, (), "k_elem_fused", "mfma"),
    ("product: fused (one launch for all groups)\n" + CHOSEN, (), "k_elem_fused", "mfma"),
    ("product: sum-factorised (one launch for all groups)\n" + ALL, ((1, 2), (2, 2)), "k_elem_factored",
     "fp64 vector fma"),
    ("product: one launch for the sum-factorised groups, one for each other group\n" + CHOSEN, ((2, 2),),
     "k_elem_factored", "fp64 vector fma / mfma"),
    ("product: one launch per group\n" + ALL.replace("-3", "1"), (), "k_elem_mfma", "mfma"),
])
def test_product_flops_and_kernel(report, factored, kernel, bound):
    prs = [P.uniform_random(3, 2, 1, 2, seed=1), P.uniform_random(4, 2, 2, 2, seed=2)]
    shapes, fused = bench.tile_shapes(report), bench.fused_product(report)
    want = sum(n * (FACTORED if g in factored else DENSE)[g] for g, n in (((1, 2), 6), ((2, 2), 8)))
    assert bench.product_flops(prs, shapes, fused) == want
    b, k = bench.product_kernel(shapes, fused)
    assert k.startswith(kernel + " ") and b == bound
