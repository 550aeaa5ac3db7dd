"""Interior blocks that hold a NaN or an infinity: every form of the inverse ends, reports
the element and leaves the others' inverses right.  (The pivot rows have to stay a
permutation of the rows, or the read-out would index by what was never written.)
Tolerance of the other elements: 1e-11 in FP64, 5e-5 in FP32, as in the forms' other
tests."""
import numpy as np
import pytest
import torch

from gpu_common import device_case, rel, to_np
from paper_1911_02366_amd import Plan, ScdgError
from workload.cases import build_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("order,modes", [(3, ("single", "blocked", "resident")), (5, ("single", "blocked", "resident")),
                                         (7, ("single", "blocked"))])
def test_nonfinite_blocks_are_reported(order, modes, precision):
    case = build_case(2, order, 1600.0, 5e-3, seed=order)
    dev = device_case(case)
    ne, ni = case.n_elem, case.n_i
    plan = Plan.from_structure(case.structure())
    for mode in modes:
        plan.set_inverse_mode(mode)
        for value in (float("nan"), float("inf"), float("-inf")):
            for row, col in ((0, 0), (ni - 1, 2), (ni // 2, ni - 1)):
                aii = dev["aii"].clone()
                aii.view(ne, ni, ni)[3, row, col] = value
                print(f"non-finite N={order} {mode} {precision} {value} at {row}, {col}", flush=True)
                plan.assemble(aii, dev["aib"], dev["abi"], dev["bb_val"])
                plan.factor(precision)
                elem, step = plan.factor_info()
                assert elem == 3 and 1 <= step <= ni
                with pytest.raises(ScdgError, match="singular interior block in element 3"):
                    plan.condense()
        dt = torch.float64 if precision == "fp64" else torch.float32
        inv = to_np(plan.export("aii_inv", ne * ni * ni, dtype=dt)).astype(np.float64).reshape(ne, ni, ni)
        for e in (2, 4):
            assert rel(inv[e], np.linalg.inv(to_np(case.aii)[e])) <= (1e-11 if precision == "fp64" else 5e-5)
    plan.close()
