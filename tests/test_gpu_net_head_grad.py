"""The head's backward kernel (its input's gradient and its own weights' from
one read), on grids of one block filled in part, of whole blocks, and of blocks
whose last pieces are missing: every layer's gradient, the head's included,
against the oracle's BF16 emulation with the tolerance of the other gradient
tests (FP32 sums of at most 1e4 terms err by far less than its 5e-3)."""
import pytest

import test_gpu_net_grad_tiles as tiles

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(8, 4, 4), (32, 8, 4), (64, 16, 4), (44, 20, 12)])
def test_head_gradient(orc, dims):
    tiles.test_gradients_on_partial_tiles(orc, dims)
