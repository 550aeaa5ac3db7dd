"""The batched products X_e = A_ii^-1 A_ib and T_e = F_e - A_bi X_e over every K
remainder and tile edge of the interior and coupling sizes (order 2 to 7: K = 5,
40, 135, 320, 625, 1080 against slabs of 16), every tile configuration, FP64 and FP32.

Reference: the float64 product of the operands as the plan holds them.  Tolerance: the
a-priori bound of a sum of K products in the format's precision u, entry by entry,
(K + 4) u (|A| |B|), with |F| added for the entries that receive a folded block."""
import pytest
import torch

from gpu_common import DEV, device_case, fold_matrices, make_plan
from workload.cases import build_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("order", [2, 3, 4, 5, 6, 7])
def test_products_at_every_slab_remainder(order, precision):
    case = build_case(2, order, 400.0, 5e-3, seed=order)
    dev = device_case(case)
    plan = make_plan(case, dev, precision)
    dt = torch.float64 if precision == "fp64" else torch.float32
    u = torch.finfo(dt).eps
    ne, ni, nc = case.n_elem, case.n_i, case.n_c
    held = lambda t, *s: t.reshape(s)[-1].to(dt).double()  # noqa: E731
    aib, abi = held(dev["aib"], ne, ni, nc), held(dev["abi"], ne, nc, ni)
    fold = torch.tensor(fold_matrices(case, [ne - 1])[ne - 1], device=DEV)
    inv = plan.export("aii_inv", ne * ni * ni, dtype=dt).reshape(ne, ni, ni)[-1].double()
    for cfg in range(9):
        print(f"gemm edges N={order} {precision} cfg={cfg}", flush=True)
        plan.set_gemm_config(cfg, cfg)
        plan.condense()
        x = plan.export("x", ne * ni * nc, dtype=dt).reshape(ne, ni, nc)[-1].double()
        t = plan.export("schur", ne * nc * nc, dtype=dt).reshape(ne, nc, nc)[-1].double()
        bound = (ni + 4) * u
        assert bool(((x - inv @ aib).abs() <= bound * (inv.abs() @ aib.abs())).all())
        assert bool(((t - (fold - abi @ x)).abs() <= bound * (abi.abs() @ x.abs() + fold.abs())).all())
    plan.close()
