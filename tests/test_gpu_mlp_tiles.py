"""FP32 network products (scdg_mlp_forward, scdg_mlp_backward) at the edges of their
tiles: K below and across a 16-deep slab, rows and columns across 16, 32 and 64,
odd row lengths, and batches that take each tile and each split of K, against the
FP64 oracle with the tolerances of test_gpu_mlp.py (2e-5 norm-wise)."""
import numpy as np
import pytest
import torch

from gpu_common import DEV, to_np
from oracle import mlp as om
from paper_1911_02366_amd.mlp import Mlp

pytestmark = pytest.mark.gpu

# n_in, hidden, layers, n_out, batch
SHAPES = [(1, 1, 1, 1, 1), (15, 16, 1, 17, 16), (33, 31, 2, 5, 65), (250, 64, 1, 125, 1030), (16, 256, 1, 260, 4097),
          (1250, 200, 1, 625, 1023), (40, 64, 0, 70, 2049)]


@pytest.mark.parametrize("shape", SHAPES)
def test_products_match_oracle(shape):
    n_in, n_h, n_l, n_out, batch = shape
    sh = (n_in, n_h, n_l, n_out)
    rng = np.random.default_rng(sum(shape))
    net = Mlp(*sh, max_batch=batch)
    w = (rng.standard_normal(net.n_params) / np.sqrt(max(n_in, n_h))).astype(np.float32)
    x = rng.standard_normal((batch, n_in)).astype(np.float32)
    dy = rng.standard_normal((batch, n_out)).astype(np.float32)
    # views that start one value into their storage: rows are aligned to nothing but a float
    on = lambda a: torch.tensor(np.concatenate([[0.0], a.reshape(-1)]).astype(np.float32), device=DEV)[1:]
    wd, xd, dyd = on(w), on(x), on(dy)
    y = net.forward(wd, xd, batch)
    dx = torch.empty_like(xd)
    dw = net.backward(wd, xd, dyd, batch, dx=dx)
    again = net.backward(wd, xd, dyd, batch)
    y_o, acts = om.forward(w, x, sh)
    dw_o, dx_o = om.backward(w, acts, dy, sh)
    close = lambda got, want: np.linalg.norm(to_np(got).astype(np.float64) - want.reshape(-1)) <= 2e-5 * np.linalg.norm(want)
    assert close(y, y_o) and close(dx, dx_o)
    for off, fi, fo, bo in om.layout(*sh)[0]:
        assert close(dw[off:off + fi * fo], dw_o[off:off + fi * fo]), ("dW", off)
        assert close(dw[bo:bo + fo], dw_o[bo:bo + fo]), ("db", bo)
    assert torch.equal(dw, again)
    net.close()
