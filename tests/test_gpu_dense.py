"""Dense LU of S (scdg_solve_condensed, solver "dense") on general matrices: pivots
inside a panel's diagonal block, whole-panel pivoting, both in one matrix, panel
remainders, and an exactly singular S.

One element whose boundary nodes all couple (A_bb full), so S = A_bb - A_bi
A_ii^-1 A_ib is any matrix the test wants; the reference is S in numpy.  The
solution is judged by its backward error ||b - S x|| / (||S||_F ||x||), which
Gaussian elimination with bounded multipliers keeps at n eps times the element
growth: 1480 x 1.1e-16 x 60 < 1e-11."""
import numpy as np
import pytest
import torch

from paper_1911_02366_amd import Plan, ScdgError

pytestmark = pytest.mark.gpu


def one_element(order, s_wanted, seed):
    """Plan and blocks of one element with S = s_wanted (A_bb takes what the Schur part removes)."""
    rng = np.random.default_rng(seed)
    p = order + 1
    nb, ni = p ** 3 - (order - 1) ** 3, 5 * (order - 1) ** 3
    n1 = 5 * nb
    aii = np.eye(ni) + 0.1 * rng.standard_normal((ni, ni)) / np.sqrt(ni)
    aib, abi = rng.standard_normal((ni, n1)) / ni, rng.standard_normal((n1, ni)) / ni
    abb = s_wanted + abi @ np.linalg.solve(aii, aib)
    plan = Plan([order], [0, nb], np.arange(nb), np.arange(nb + 1) * nb, np.tile(np.arange(nb), nb))
    t = lambda a: torch.tensor(np.ascontiguousarray(a), device="cuda")
    bb = abb.reshape(nb, 5, nb, 5).transpose(0, 2, 1, 3)
    plan.assemble(t(aii), t(aib), t(abi), t(bb))
    plan.factor("fp64")
    plan.condense()
    return plan


def wanted(kind, n, rng):
    s = rng.standard_normal((n, n))
    if kind == "dominant":
        return s / n + np.eye(n)
    if kind == "scaled_rows":                 # dominant but for rows of very different size
        return (s / n + np.eye(n)) * 10.0 ** rng.uniform(-6, 6, n)[:, None]
    if kind == "half":                        # the first panels find their pivots inside, the last ones do not
        s[: n // 2] = s[: n // 2] / n + np.eye(n)[: n // 2]
        return s
    if kind == "antidiagonal":                # every pivot lies in another panel
        return s / n + np.eye(n)[::-1]
    return s


@pytest.mark.parametrize("order", [2, 3, 7])   # n1 = 130, 280, 1480: panels of 64 with remainders 2, 24, 8
@pytest.mark.parametrize("kind", ["dominant", "scaled_rows", "random", "half", "antidiagonal"])
def test_dense_lu_backward_error(order, kind):
    n = 5 * ((order + 1) ** 3 - (order - 1) ** 3)
    rng = np.random.default_rng(order)
    s = wanted(kind, n, rng)
    plan = one_element(order, s, 1)
    for rhs in range(2):                       # the second solve reuses the factors
        b = rng.standard_normal(n)
        x, info = plan.solve_condensed(torch.tensor(b, device="cuda"), solver="dense")
        x = x.cpu().numpy()
        assert info["solver_used"] == 1
        err = np.linalg.norm((b - s @ x) / np.abs(s).max(axis=1)) / np.linalg.norm(x)
        err /= np.linalg.norm(s / np.abs(s).max(axis=1)[:, None])
        assert err <= 1e-11, (order, kind, rhs, err)
    plan.close()


def test_dense_lu_singular():
    n = 130
    rng = np.random.default_rng(3)
    s = rng.standard_normal((n, n))
    plan = one_element(2, s, 1)
    nb = n // 5
    zero = np.zeros((nb, nb, 5, 5))            # A_bb = 0 and A_bi = 0: S = 0 exactly
    t = lambda a: torch.tensor(np.ascontiguousarray(a), device="cuda")
    plan.assemble(t(np.eye(5)), t(np.zeros((5, n))), t(np.zeros((n, 5))), t(zero))
    plan.factor("fp64")
    plan.condense()
    with pytest.raises(ScdgError, match="zero pivot in the dense LU of S at step 1"):
        plan.solve_condensed(torch.ones(n, dtype=torch.float64, device="cuda"), solver="dense")
    plan.close()
