"""GMRES on a system whose S holds a NaN or an infinity ends with SCDG_ERR_NONFINITE in
every mode and form of the products, never as a success with a NaN vector, and the plan
solves the sound system afterwards."""
import numpy as np
import pytest
import torch

from gpu_common import device_case, rel, to_np
from paper_1911_02366_amd import Plan
from workload.cases import build_case

pytestmark = pytest.mark.gpu
NONFINITE = -7


@pytest.mark.parametrize("value", [float("nan"), float("inf")])
@pytest.mark.parametrize("precond", [0, 1, 2])
@pytest.mark.parametrize("mode", ["host", "device", "graph"])
def test_gmres_reports_nonfinite(mode, precond, value):
    case = build_case(2, 3, 100.0, 1e-2, seed=1)
    dev = device_case(case)
    plan = Plan.from_structure(case.structure())
    plan.set_krylov_mode(mode)
    opts = dict(solver="gmres", restart=30, precond=precond, tol=1e-10)
    sound, bad = dev["bb_val"], dev["bb_val"].clone()
    bad.view(-1)[7] = value
    for schur in ("assembled", "matrix_free"):
        plan.set_schur_mode(schur)
        for bb in (bad, sound):
            plan.assemble(dev["aii"], dev["aib"], dev["abi"], bb)
            plan.factor("fp64")
            plan.condense()
            bs = plan.condense_rhs(dev["b"])
            for x0 in (None, bs.clone()):
                x, info = plan.solve_condensed(bs, x0=x0, check=False, **opts)
                print(f"gmres {mode} precond {precond} {schur} {value} status {info['status']}", flush=True)
                if bb is bad:
                    assert info["status"] == NONFINITE
                else:
                    assert info["status"] == 0
                    assert rel(to_np(plan.schur_apply(x)), to_np(bs)) <= 1e-9
    plan.close()
