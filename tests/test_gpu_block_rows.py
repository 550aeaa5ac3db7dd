"""Block-row products over the row lengths that the couplings of orders 2 to 7 have
(trips of 24 blocks, a last one of 12 or fewer, rows of one trip): the full A_bb, A_ib
and A_bi rows of the block-sparse form and the A_bb remainder of the assembled form.

The three forms of the Schur product are sums of the same terms: FP64 agrees to 1e-12
of the largest entry, FP32 blocks (products summed in FP64) to 2e-5, as in the forms'
other tests; the full residual, whose A_bb product is the same kernel's, is compared
with a dense product in float64."""
import pytest
import torch

from gpu_common import DEV, device_case, oracle_arrays, oracle_matrix, make_plan
from workload.cases import build_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("order", [2, 3, 4, 5, 6, 7])
def test_forms_agree_at_every_row_length(order, precision):
    print(f"block rows N={order} {precision}", flush=True)
    case = build_case(2, order, 800.0, 5e-3, seed=order)
    plan = make_plan(case, device_case(case), precision)
    gen = torch.Generator(device=DEV).manual_seed(order)
    x = torch.randn(case.n1, dtype=torch.float64, device=DEV, generator=gen)
    y = {}
    for mode in ("assembled", "matrix_free", "matrix_free_sparse"):
        plan.set_schur_mode(mode)
        plan.condense()
        y[mode] = plan.schur_apply(x).clone()
    big = float(y["assembled"].abs().max())
    for mode in ("matrix_free", "matrix_free_sparse"):
        err = float((y[mode] - y["assembled"]).abs().max()) / big
        print(f"  {mode} {err:.1e}", flush=True)
        assert err <= (1e-12 if precision == "fp64" else 2e-5)
    plan.close()


@pytest.mark.parametrize("order", [2, 3, 4])
def test_residual_of_the_full_system(order):
    case = build_case(2, order, 800.0, 5e-3, seed=order)
    dev = device_case(case)
    plan = make_plan(case, dev)
    gen = torch.Generator(device=DEV).manual_seed(order)
    x = torch.randn(case.n_dof, dtype=torch.float64, device=DEV, generator=gen)
    r = torch.empty_like(x)
    plan.residual(dev["b"], x, r)
    want = dev["b"].cpu().numpy() - oracle_matrix(oracle_arrays(case)) @ x.cpu().numpy()
    assert abs(r.cpu().numpy() - want).max() <= 1e-12 * abs(want).max()
    plan.close()
