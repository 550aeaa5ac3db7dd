"""On curved elements each element takes a face's flux along its own face vector, so that a
constant flux cancels in its sums by the metric identity of its own terms, whatever its
neighbours' terms round to.

One corner node is moved by 1e-3.  The metric terms are formed from positions relative to
an element's first node, so those of the eight elements around the corner change, also in
the last digits on faces that did not move.  With a constant state the mass residual
(no viscous part, no jump) of every other element stays the same to the last bit."""
import numpy as np
import pytest
import torch

from gpu_common import DEV, to_np
from paper_1911_02366_amd.dg import DgResidual
from workload import dgsem as wd
from workload.physics import FlowParams

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["sine", "skew"])
@pytest.mark.parametrize("order", [2, 3, 4, 5, 6, 7])
def test_mass_residual_of_a_constant_state_is_local(order, kind):
    k, p = 3, order + 1
    mesh, prm = wd.Mesh(k, order), FlowParams(mach=0.1, reynolds=1600.0)
    xyz = wd.curved_node_coordinates(mesh, kind=kind).copy()
    q = torch.tensor(wd.uniform_state(mesh, prm).reshape(-1), device=DEV)
    dg = DgResidual(k, order, mach=prm.mach, reynolds=prm.reynolds)

    def mass_residual():
        dg.set_geometry(xyz)
        return to_np(dg.residual(q)).reshape(k, k, k, p ** 3, 5)[..., 0]

    before = mass_residual()
    away = np.ones((k, k, k), bool)
    for c in np.ndindex(2, 2, 2):                          # the corner of element (1, 1, 1) in its eight elements
        xyz[c + tuple(order if i == 0 else 0 for i in c)] += [1e-3, -7e-4, 5e-4]
        away[c] = False
    after = mass_residual()
    print(f"mass residual N={order} {kind}: {np.abs(before).max():.1e}, near the corner {np.abs(after - before).max():.1e}", flush=True)
    assert not np.array_equal(before[~away], after[~away])
    np.testing.assert_array_equal(before[away], after[away])
    dg.close()
