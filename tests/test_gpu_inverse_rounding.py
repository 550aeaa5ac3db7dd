"""Rounding of the blocked inverse: its updates C += A B add the sum of products to C
once, so that a product is rounded at its own size and not at C's, and the inverse is no
further from the exact one than the single-kernel form's (whole-column pivots, panels of
16 to 32 columns whose updates do the same), on interior blocks of the flow.  The exact
inverse is LAPACK's, refined by one Newton step with the residual in extended precision
(off by its square, under 1e-20)."""
import numpy as np
import pytest
import torch

from gpu_common import device_case, to_np
from paper_1911_02366_amd import Plan
from workload.cases import build_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("order,dt", [(5, 5e-3), (6, 5e-3), (6, 1e-2)])
def test_blocked_inverse_is_no_further_off(order, dt, precision):
    case = build_case(2, order, 1600.0, dt, seed=order)
    dev = device_case(case)
    ne, ni = case.n_elem, case.n_i
    a = to_np(dev["aii"]).reshape(ne, ni, ni)[0]
    x = np.linalg.inv(a)
    res = (np.eye(ni, dtype=np.longdouble) - a.astype(np.longdouble) @ x.astype(np.longdouble)).astype(np.float64)
    step = x @ res
    plan = Plan.from_structure(case.structure())
    plan.assemble(dev["aii"], dev["aib"], dev["abi"], dev["bb_val"])
    err = {}
    for mode in ("single", "blocked"):
        plan.set_inverse_mode(mode)
        plan.factor(precision)
        dtype = torch.float64 if precision == "fp64" else torch.float32
        inv = to_np(plan.export("aii_inv", ne * ni * ni, dtype=dtype)).astype(np.float64).reshape(ne, ni, ni)[0]
        err[mode] = np.linalg.norm((inv - x) - step) / np.linalg.norm(x)
    print(f"inverse rounding N={order} dt={dt} {precision}: {err}", flush=True)
    assert err["blocked"] <= err["single"]
    plan.close()
