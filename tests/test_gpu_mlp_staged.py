"""FP32 network products large enough for tiles staged in LDS: a layer's from 1024 tiles
and K = 768 on, a gradient's from 512, one step on either side of the lines, against the
FP64 oracle with the tolerances of the network's other tests; the bias gradients come
from a launch of their own beside the staged dW."""
import pytest

import test_gpu_mlp_tiles as tiles

pytestmark = pytest.mark.gpu

# n_in, hidden, layers, n_out, batch: all products staged (K remainders 13, 1 and 1); dZ
# of 516 tiles beside small dW; dZ of 508; layers of 1056 tiles with K = 767 and 769
SHAPES = [(1501, 1409, 1, 65, 4097), (100, 256, 1, 30, 8193), (100, 256, 1, 30, 8100), (767, 1025, 1, 9, 3969),
          (769, 1025, 1, 9, 3969)]


@pytest.mark.parametrize("shape", SHAPES)
def test_staged_products_match_oracle(shape):
    tiles.test_products_match_oracle(shape)
