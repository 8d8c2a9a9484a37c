"""The first layer's weight gradient with more blocks than compute units (from
1024 tiles of 16 x 4 x 2 voxels; rows of 4 voxels keep the grids small): 288 and
512 blocks, the second with a remainder of tiles.  Against the oracle's BF16
emulation, with the tolerance of the other gradient tests."""
import pytest

import test_gpu_net_grad_tiles as tiles

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(4, 72, 128), (4, 136, 124)])
def test_first_layer_blocks(orc, dims):
    tiles.test_gradients_on_partial_tiles(orc, dims)
