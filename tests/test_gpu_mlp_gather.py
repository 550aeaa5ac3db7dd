"""Row gathers are exact at odd widths on either side of 256 (values a thread below, a
workgroup a row from there on), with one row and with counts that leave a part of a
workgroup, and write nothing past the last row."""
import pytest
import torch

from gpu_common import DEV
from paper_1911_02366_amd.mlp import Mlp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("width", [1, 5, 64, 135, 255, 256, 257, 1250])
def test_gather_rows(width):
    net = Mlp(4, 4, 1, 4, max_batch=1)
    gen = torch.Generator(device=DEV).manual_seed(width)
    src = torch.randn(1003, width, device=DEV, generator=gen)
    for count in (1, 255, 1003):
        idx = torch.randint(0, 1003, (count,), device=DEV, generator=gen, dtype=torch.int32)
        guard = torch.full((count * width + 64,), 7.0, device=DEV)
        net.gather(src.reshape(-1), width, idx, count, guard)
        assert torch.equal(guard[:count * width].reshape(count, width), src[idx.long()])
        assert bool((guard[count * width:] == 7.0).all())
    net.close()
