"""Dense LU of S on well-conditioned matrices whose entries grow from panel to panel when
the pivots stay inside the 64 x 64 diagonal blocks (the coupled rows of
test_gpu_inverse_growth.py): every multiplier is 1/d, and the last columns grow by 1/d
a panel.  Partial pivoting meets no growth.  And matrices with a NaN or an infinity, which are reported.

Tolerance on the solution's relative error: n eps cond, 1480 x 1.1e-16 x 30 < 1e-11."""
import numpy as np
import pytest
import torch

from paper_1911_02366_amd import ScdgError
from test_gpu_dense import one_element
from test_gpu_inverse_growth import coupled

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order", [2, 3, 5, 7])            # n1 = 130, 280, 760, 1480
@pytest.mark.parametrize("d", [1 / 1.3, 1 / 2, 1 / 3.9, 1 / 7.5])
def test_dense_lu_growth(order, d):
    n = 5 * ((order + 1) ** 3 - (order - 1) ** 3)
    s = coupled(n, d) * 10.0 ** np.random.default_rng(2).uniform(-3, 3, n)[:, None]
    plan = one_element(order, s, 1)
    rng = np.random.default_rng(order)
    for rhs in range(2):
        want = rng.standard_normal(n)
        x, info = plan.solve_condensed(torch.tensor(s @ want, device="cuda"), solver="dense")
        assert info["solver_used"] == 1
        err = np.linalg.norm(x.cpu().numpy() - want) / np.linalg.norm(want)
        print(f"dense growth n={n} d={d:.3f}: {err:.1e}", flush=True)
        assert err <= 1e-11
    plan.close()


@pytest.mark.parametrize("value", [float("nan"), float("inf")])
@pytest.mark.parametrize("at", [(0, 0), (70, 3), (129, 129)])
def test_dense_lu_nonfinite(at, value):
    s = coupled(130, 2.0)
    plan = one_element(2, s, 1)
    t = lambda a: torch.tensor(np.ascontiguousarray(a), device="cuda")
    s[at] = value
    plan.assemble(t(np.eye(5)), t(np.zeros((5, 130))), t(np.zeros((130, 5))),
                  t(s.reshape(26, 5, 26, 5).transpose(0, 2, 1, 3)))
    plan.factor("fp64")
    plan.condense()
    print(f"dense non-finite {value} at {at}", flush=True)
    with pytest.raises(ScdgError, match="zero pivot in the dense LU of S"):
        plan.solve_condensed(torch.ones(130, dtype=torch.float64, device="cuda"), solver="dense")
    plan.close()
