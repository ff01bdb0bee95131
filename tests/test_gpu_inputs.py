"""Single products and sensitivities, whose inputs one launch prepares: in
place (y = x, y overlapping the end of x) and for exponents beside q = 3, for
which the power is a product.

Tolerance (written here): in-place results equal the separate call's to the
bit (the same arithmetic); against the oracle's moduli 1e-12 of the largest
value, a few hundred FP64 roundings."""

import numpy as np
import pytest
import torch

from oracle.mechanism import bilinear_sensitivity
from oracle import oracle_solve
from paper_1811_09821_amd import problems as P

pytestmark = pytest.mark.gpu


def mto():
    from paper_1811_09821_amd import mto as m

    return m


@pytest.mark.parametrize("name", ["apply_stiffness", "apply_stiffness_noalloc"])
def test_product_in_place(cuda, name):
    import ctypes

    m = mto()
    pr = P.small_mixed(13, 7, seed=5, n_loads=2)
    plan = m.Plan(pr)
    n = plan.info["n_u"]
    rho = torch.tensor(pr.rho, device=cuda)
    x = torch.randn(n, dtype=torch.float64, device=cuda, generator=torch.Generator(device=cuda).manual_seed(1))
    fn = getattr(m._lib, "mto_" + name)

    def call(r, a, b):
        rc = fn(plan.handle, ctypes.c_void_p(r), ctypes.c_void_p(a), ctypes.c_void_p(b),
                ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
        assert rc == 0
        torch.cuda.synchronize()

    y = torch.full((n,), 7.0, dtype=torch.float64, device=cuda)
    call(rho.data_ptr(), x.data_ptr(), y.data_ptr())
    z = x.clone()
    call(rho.data_ptr(), z.data_ptr(), z.data_ptr())
    assert torch.equal(y, z)
    both = torch.cat([x, torch.zeros(5, dtype=torch.float64, device=cuda)])  # y overlaps the end of x
    call(rho.data_ptr(), both.data_ptr(), both[5:].data_ptr())
    assert torch.equal(y, both[5:])


@pytest.mark.parametrize("q", [1.0, 2.0, 3.0, 3.5, 4.0])
def test_penalty_exponents(cuda, q):
    pr = P.uniform_random(9, 5, 2, 3, seed=6, lo=0.0, hi=1.0)
    o = oracle_solve(**pr.oracle_args())
    g = mto().Plan(pr, q=q).sensitivity(torch.tensor(pr.rho, device=cuda), torch.tensor(o["u"].ravel(), device=cuda))
    ref = bilinear_sensitivity(pr.nelx, pr.nely, pr.p, pr.d, pr.rho, o["u"][0], o["u"][0], q=q)
    assert np.abs(g.cpu().numpy() - ref).max() <= 1e-12 * np.abs(ref).max()
