"""The blocked inverse on well-conditioned blocks whose entries grow from one 64 x 64
diagonal block to the next when the pivots stay inside them: rows r, r + 64, r + 128, ..
are coupled for each r < 64, with d on the diagonal, -1 below it and 1 in the last of
the coupled columns.  Multipliers inside a block are 1/d, the last columns grow by 1/d a
block (or, with d >= 1, by 2), and the condition number stays below 30; partial pivoting
over whole columns meets no growth at all for d < 1.

Tolerance: the error of an inverse by elimination is bounded by n eps cond times the
growth; 1080 x 1.1e-16 x 30 x 8 < 1e-10 and, with the random signs of rounding (the
square root of n), 1e-11 and in FP32 5e-5 as in the blocked form's other tests."""
import numpy as np
import pytest
import torch

from gpu_common import DEV, rel, to_np
from paper_1911_02366_amd import Plan

pytestmark = pytest.mark.gpu


def coupled(n, d):
    """The matrix of the header and its condition number."""
    a = np.eye(n) * d
    for r in range(min(64, n)):
        rows = np.arange(r, n, 64)
        a[rows[1:], rows[:-1]] = -1.0
        a[rows, rows[-1]] = 1.0
    return a


def one_element(order, aii):
    """A plan of one element with interior block aii, nothing coupled to it."""
    nb, ni = (order + 1) ** 3 - (order - 1) ** 3, 5 * (order - 1) ** 3
    plan = Plan([order], [0, nb], np.arange(nb), np.arange(nb + 1), np.arange(nb))
    zero = torch.zeros(ni * 5 * nb, dtype=torch.float64, device=DEV)
    bb = torch.eye(5, dtype=torch.float64, device=DEV).repeat(nb, 1, 1).reshape(-1)
    plan.set_inverse_mode("blocked")
    plan.assemble(torch.tensor(aii, device=DEV).reshape(-1), zero, zero, bb)
    return plan


@pytest.mark.parametrize("order", [5, 6, 7])               # n_i = 320, 625, 1080
@pytest.mark.parametrize("d", [1.0, 1 / 1.3, 1 / 2, 1 / 3.9, 1 / 7.5, 1 / 30])
def test_blocked_inverse_growth(order, d):
    ni = 5 * (order - 1) ** 3
    a = coupled(ni, d)
    ref = np.linalg.inv(a)
    print(f"inverse growth N={order} d={d:.3f} cond {np.linalg.cond(a):.1f}", flush=True)
    plan = one_element(order, a)
    for precision in ("fp64", "fp32"):
        plan.factor(precision)
        assert plan.factor_info()[0] == -1
        dt = torch.float64 if precision == "fp64" else torch.float32
        err = rel(to_np(plan.export("aii_inv", ni * ni, dtype=dt)).astype(np.float64).reshape(ni, ni), ref)
        print(f"  {precision}: {err:.1e}", flush=True)
        assert err <= (1e-11 if precision == "fp64" else 5e-5)
    plan.close()
