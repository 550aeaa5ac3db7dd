"""GMRES cycles at the edges of their launches: fewer unknowns than workgroups have
threads, basis sizes that take each register bucket of the Gram-Schmidt kernels
and the 32-rows-at-a-time form past 32 (restart up to 63), every preconditioner, an
iteration limit inside a cycle, a start at the solution.  The reference is the dense
solve of S by the oracle; the stopping test is on the true residual, so a solve to
1e-12 is within cond(S) 1e-12 of it, 2.5e-9 in the worst direction (cond 2.5e3) and a tenth
of that in a general one.  (Restart 1 stalls at 0.2 on this S in exact arithmetic too.)"""
import numpy as np
import pytest
import torch

import oracle
from gpu_common import DEV, device_case, make_plan, oracle_arrays, rel, to_np
from workload.cases import build_case

pytestmark = pytest.mark.gpu


def _system(k, n, dt):
    case = build_case(k, n, 1600.0, dt, seed=3)
    d = oracle_arrays(case)
    s = oracle.condensed_matrix_dense(d["c_ptr"], d["c_node"], d["bb_rowptr"], d["bb_col"], d["bb_val"], d["aii"],
                                      d["aib"], d["abi"])
    return make_plan(case, device_case(case)), s


@pytest.mark.parametrize("mode", ["host", "device", "graph"])
@pytest.mark.parametrize("restart", [3, 9, 31, 32, 33, 63])
def test_restart_lengths(mode, restart):
    plan, s = _system(2, 2, 5e-2)                  # n1 = 1040
    plan.set_krylov_mode(mode)
    rng = np.random.default_rng(restart)
    for rep in range(2):
        x = rng.standard_normal(len(s))
        bs = torch.tensor(s @ x, device=DEV)
        qb, info = plan.solve_condensed(bs, solver="gmres", tol=1e-12, restart=restart, max_iters=3000)
        assert rel(to_np(qb), x) <= 1e-9, (mode, restart, info)
        assert info["rel_res_S"] <= 1e-12 and info["restarts"] >= (info["iters"] + restart - 1) // restart
    plan.close()


@pytest.mark.parametrize("precond", [0, 1, 2])
def test_preconditioners_limits_and_guess(precond):
    plan, s = _system(2, 3, 2e-2)                  # n1 = 2240
    x = np.random.default_rng(5).standard_normal(len(s))
    bs = torch.tensor(s @ x, device=DEV)
    qb, info = plan.solve_condensed(bs, solver="gmres", tol=1e-12, restart=20, precond=precond, max_iters=2000)
    assert rel(to_np(qb), x) <= 1e-9, (precond, info)
    # an iteration limit inside the second cycle: the partial solution and its true residual
    part, lim = plan.solve_condensed(bs, solver="gmres", tol=1e-14, restart=4, precond=precond, max_iters=6, check=False)
    assert lim["iters"] == 6 and lim["restarts"] == 2 and lim["status"] == -6
    res = np.linalg.norm(s @ (x - to_np(part))) / np.linalg.norm(s @ x)
    assert abs(res - lim["rel_res_S"]) <= 1e-10
    # a start at the solution needs no iteration, a start far from it is dropped
    _, at = plan.solve_condensed(bs, x0=qb, solver="gmres", tol=1e-10, precond=precond)
    assert at["iters"] == 0 and at["rel_res_guess"] <= 1e-11
    far, off = plan.solve_condensed(bs, x0=100.0 * qb, solver="gmres", tol=1e-12, precond=precond, max_iters=2000)
    assert off["guess_rejected"] == 1 and rel(to_np(far), x) <= 1e-9
    plan.close()
