"""The blocked inverse where its pivots stay inside 64 x 64 diagonal blocks and where
they cannot: plain interior blocks, rows scaled by powers of two over 2^24 (the
pivot choice sees scaled rows, the values are not scaled), and rows rolled by half
the block, whose diagonal blocks hold no usable pivots (the whole-column form).

Sizes: n_i = 40 (part of one block), 135 (two blocks and 7), 320 (five), 625 (a last
block of 49), 1080 (seventeen, the last of 56).  Tolerance: that of the blocked form's
other tests, 1e-11 per element in FP64 and 5e-5 in FP32, against LAPACK's inverse;
scaled columns are compared after the exact unscaling."""
import numpy as np
import pytest
import torch

from gpu_common import DEV, device_case, rel, to_np
from paper_1911_02366_amd import Plan
from workload.cases import build_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("kind", ["plain", "scaled", "rolled"])
@pytest.mark.parametrize("order", [3, 4, 5, 6, 7])
def test_blocked_inverse_pivots(order, kind, precision):
    print(f"inverse pivots N={order} {kind} {precision}", flush=True)
    case = build_case(2, order, 1600.0, 5e-3, seed=order)
    dev = device_case(case)
    ne, ni = case.n_elem, case.n_i
    a = to_np(dev["aii"]).reshape(ne, ni, ni)
    scale = np.ones(ni)
    if kind == "scaled":
        scale = 2.0 ** np.random.default_rng(order).integers(-12, 13, ni)
        a = a * scale[None, :, None]
    elif kind == "rolled":
        a = np.roll(a, ni // 2, axis=1)
    dev["aii"] = torch.tensor(np.ascontiguousarray(a).reshape(-1), device=DEV)
    plan = Plan.from_structure(case.structure())
    plan.set_inverse_mode("blocked")
    plan.assemble(dev["aii"], dev["aib"], dev["abi"], dev["bb_val"])
    plan.factor(precision)
    assert plan.factor_info()[0] == -1
    dt = torch.float64 if precision == "fp64" else torch.float32
    inv = to_np(plan.export("aii_inv", ne * ni * ni, dtype=dt)).astype(np.float64).reshape(ne, ni, ni)
    for e in (0, ne - 1):
        err = rel(inv[e] * scale[None, :], np.linalg.inv(a[e] / scale[:, None]))
        print(f"  element {e}: {err:.1e}", flush=True)
        assert err <= (1e-11 if precision == "fp64" else 5e-5)
    plan.close()
