"""Every order the residual's kernels are built for (2 to 7), each face form
(Bassi-Rebay 1, SIPG, curved), against the oracle: the residual, its exported
gradient and the Newton-matrix product, which the two-field lift feeds. Three
elements a direction make every neighbour distinct and the pair count
(27 p^2) ragged against 256 threads at all orders.

Tolerance: as for the residual's other oracle tests, 1e-11 of the largest entry:
both sides are exact to rounding and sum the same FP64 terms in different orders."""
import numpy as np
import pytest
import torch

from gpu_common import DEV, to_np
from oracle import dgsem as od
from paper_1911_02366_amd import DgResidual
from workload import dgsem as wd
from workload.physics import FlowParams

pytestmark = pytest.mark.gpu

RTOL = 1e-11


def _rel(got, want):
    return float(np.abs(got.reshape(-1) - want.reshape(-1)).max() / np.abs(want).max())


@pytest.mark.parametrize("form", ["br1", "sipg", "curved"])
@pytest.mark.parametrize("n", [2, 3, 4, 5, 6, 7])
def test_every_order_and_face_form(n, form):
    print(f"dg orders N={n} {form}", flush=True)
    k, mach, re = 3, 0.2, 400.0
    mesh, grid, flow = wd.Mesh(k, n), od.Grid(k, n), od.Flow(mach, re)
    xyz = wd.curved_node_coordinates(mesh, 0.05, "skew") if form == "curved" else None
    q = wd.taylor_green_state(mesh, FlowParams(mach, re), n, coords=xyz)
    qs = wd.taylor_green_state(mesh, FlowParams(mach, re), n + 20, coords=xyz)
    v = np.random.default_rng(n).standard_normal(q.shape)
    dg = DgResidual(k, n, mach=mach, reynolds=re, viscous="sipg" if form == "sipg" else "br1")
    if form == "curved":
        dg.set_geometry(xyz)
        ja, jac = od.metric_terms(xyz, grid)
        want = (od.residual_curved(q, grid, flow, ja, jac, qs, 0.01), od.lifted_gradient_curved(q, grid, ja, jac),
                od.jacobian_apply_curved(q, v, grid, flow, ja, jac, 0.25))
    else:
        want = (od.residual(q, grid, flow, qs, 0.01, viscous=form), od.lifted_gradient(q, grid),
                od.jacobian_apply(q, v, grid, flow, 0.25, viscous=form))
    qd, qsd, vd = (torch.tensor(a.reshape(-1), device=DEV) for a in (q, qs, v))
    r = to_np(dg.residual(qd, qsd, 100.0))
    g = to_np(dg.gradient())
    av = to_np(dg.jacobian_apply(qd, vd, 4.0))
    errs = [_rel(a, b) for a, b in zip((r, g, av), want)]
    print("  residual %.1e gradient %.1e product %.1e" % tuple(errs), flush=True)
    assert max(errs) <= RTOL
    dg.close()
