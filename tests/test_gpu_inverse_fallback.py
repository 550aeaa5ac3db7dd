"""The blocked inverse element by element: which elements take the whole-column form, and
a captured factor replayed on blocks that take the other form than at capture.

Rows rolled by half the block (as in the diagonal form's tests) leave the diagonal
blocks without usable pivots; plain and row-scaled blocks keep the diagonal form.
Sizes: n_i = 135 (one outer panel of two blocks), 625 and 1080 (five and nine outer
panels), and elements of orders 3 to 7 in one plan.  Tolerance: 1e-11 in FP64 and 5e-5
in FP32, as in the blocked form's other tests."""
import numpy as np
import pytest
import torch

from gpu_common import DEV, device_case, rel, to_np
from paper_1911_02366_amd import Plan
from test_gpu_inverse_growth import coupled
from workload.cases import build_case

pytestmark = pytest.mark.gpu
TOL = {"fp64": 1e-11, "fp32": 5e-5}


def inverse_errors(plan, blocks, precision):
    dt = torch.float64 if precision == "fp64" else torch.float32
    inv = to_np(plan.export("aii_inv", sum(a.size for a in blocks), dtype=dt)).astype(np.float64)
    out, off = [], 0
    for a in blocks:
        out.append(rel(inv[off:off + a.size].reshape(a.shape), np.linalg.inv(a)))
        off += a.size
    return out


def flat(blocks):
    return torch.tensor(np.concatenate([a.reshape(-1) for a in blocks]), device=DEV)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("order", [4, 6, 7])
def test_elements_choose_their_form(order, precision):
    case = build_case(2, order, 1600.0, 5e-3, seed=order)
    dev = device_case(case)
    ne, ni = case.n_elem, case.n_i
    plain = [a for a in to_np(dev["aii"]).reshape(ne, ni, ni)]
    scale = 2.0 ** np.random.default_rng(order).integers(-12, 13, ni)
    some = list(plain)
    some[1], some[2], some[6] = np.roll(plain[1], ni // 2, axis=0), coupled(ni, 1 / 7.5), np.roll(plain[6], ni // 2, axis=0)
    plan = Plan.from_structure(case.structure())
    plan.set_inverse_mode("blocked")
    for name, blocks, whole in (("plain", plain, 0), ("some", some, 3), ("scaled", [a * scale[:, None] for a in plain], 0),
                                ("rolled", [np.roll(a, ni // 2, axis=0) for a in plain], ne)):
        plan.assemble(flat(blocks), dev["aib"], dev["abi"], dev["bb_val"])
        plan.factor(precision)
        print(f"N={order} {precision} {name}: {plan.inverse_whole_column()} elements over whole columns", flush=True)
        assert plan.factor_info()[0] == -1
        assert plan.inverse_whole_column() == whole
        if name != "scaled":
            assert max(inverse_errors(plan, blocks, precision)) <= TOL[precision]
    plan.close()


def uneven(orders):
    """A plan of uncoupled elements and the sizes of their interior blocks."""
    nb = [(n + 1) ** 3 - (n - 1) ** 3 for n in orders]
    ni = [5 * (n - 1) ** 3 for n in orders]
    plan = Plan(orders, np.concatenate([[0], np.cumsum(nb)]), np.arange(sum(nb)), np.arange(sum(nb) + 1), np.arange(sum(nb)))
    zero = torch.zeros(sum(5 * i * b for i, b in zip(ni, nb)), dtype=torch.float64, device=DEV)
    bb = torch.eye(5, dtype=torch.float64, device=DEV).repeat(sum(nb), 1, 1).reshape(-1)
    plan.set_inverse_mode("blocked")
    return plan, ni, zero, bb


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_captured_factor(precision):
    plan, ni, zero, bb = uneven([3, 7, 4, 6, 5, 7])
    rng = np.random.default_rng(5)
    good = [np.eye(n) + 0.5 * rng.standard_normal((n, n)) / np.sqrt(n) for n in ni]
    rolled = [np.roll(a, len(a) // 2, axis=0) for a in good]
    mixed = [r if e % 2 else g for e, (g, r) in enumerate(zip(good, rolled))]
    singular = list(good)
    singular[3] = good[3].copy()
    singular[3][:, 100] = 0.0
    aii = flat(good)
    stream = torch.cuda.Stream()
    plan.set_stream(stream)
    with torch.cuda.stream(stream):
        plan.assemble(aii, zero, zero, bb)
        plan.factor(precision)                  # builds the plan's work lists
        stream.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            plan.factor(precision)
        for name, blocks in (("good", good), ("mixed", mixed), ("singular", singular), ("rolled", rolled), ("good", good)):
            aii.copy_(flat(blocks))
            graph.replay()
            stream.synchronize()
            print(f"captured {precision} {name}: {plan.inverse_whole_column()} over whole columns", flush=True)
            if name == "singular":
                assert plan.factor_info()[0] == 3 and plan.inverse_whole_column() == 1
                continue
            assert plan.factor_info()[0] == -1
            errs = inverse_errors(plan, blocks, precision)
            plan.factor(precision)              # eager work between the replays, the same answer
            assert errs == inverse_errors(plan, blocks, precision)
            assert max(errs) <= TOL[precision]
    plan.close()
