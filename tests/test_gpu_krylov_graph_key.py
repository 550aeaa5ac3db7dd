"""A captured GMRES cycle is captured again when any of its buffers has moved: a longer
restart in another mode reallocates the cycle's state, and factoring in FP64 between two
FP32 solves reallocates the factors and blocks.  Solutions against LAPACK's of the
assembled S (from the oracle's blocks), 1e-9 (the tolerance asked for is 1e-11 in FP64;
with FP32 factors S itself is off by a few 1e-6, so there 1e-4)."""
import numpy as np
import pytest

from gpu_common import device_case, rel, to_np
from paper_1911_02366_amd import Plan
from workload.cases import build_case

pytestmark = pytest.mark.gpu


def dense_s(case):
    s = np.zeros((case.n1, case.n1))
    bb, blocks = to_np(case.bb_val), [to_np(x) for x in (case.aii, case.aib, case.abi)]
    for g in range(case.n_bnodes):
        for b in range(case.bb_rowptr[g], case.bb_rowptr[g + 1]):
            s[5 * g:5 * g + 5, 5 * case.bb_col[b]:5 * case.bb_col[b] + 5] += bb[b]
    for e in range(case.n_elem):
        at = (5 * case.c_node[case.c_ptr[e]:case.c_ptr[e + 1], None] + np.arange(5)).reshape(-1)
        aii, aib, abi = (x[e] for x in blocks)
        s[np.ix_(at, at)] -= abi @ np.linalg.solve(aii, aib)
    return s


@pytest.mark.parametrize("schur", ["assembled", "matrix_free", "matrix_free_sparse"])
def test_graph_after_its_buffers_moved(schur):
    case = build_case(2, 3, 100.0, 1e-2, seed=2)
    dev = device_case(case)
    s = dense_s(case)
    plan = Plan.from_structure(case.structure())
    plan.set_schur_mode(schur)
    plan.assemble(dev["aii"], dev["aib"], dev["abi"], dev["bb_val"])

    def solve(mode, precision, restart):
        plan.set_krylov_mode(mode)
        plan.factor(precision)
        plan.condense()
        bs = plan.condense_rhs(dev["b"])
        x, info = plan.solve_condensed(bs, solver="gmres", restart=restart, precond=1,
                                       tol=1e-11 if precision == "fp64" else 1e-7)
        err = rel(to_np(x), np.linalg.solve(s, to_np(bs)))
        print(f"{schur} {mode} {precision} restart {restart}: {err:.1e}", flush=True)
        assert info["status"] == 0 and err <= (1e-9 if precision == "fp64" else 1e-4)

    for restart in (20, 40, 20, 63, 20):                    # graph, longer in another mode, graph again
        solve("graph" if restart == 20 else "device", "fp64", restart)
    for mode, precision in (("graph", "fp32"), ("host", "fp64"), ("graph", "fp32"), ("graph", "fp64"), ("graph", "fp32")):
        solve(mode, precision, 20)
    plan.close()
