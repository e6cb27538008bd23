"""GPU: products whose reduction is shorter than a K tile or a few of them, at
the edges of the rules that give them a path of their own, through the pre-LSTM
layer; bounds as for its other shapes."""
import pytest

import tests.test_gpu_gemm_tiles as tiles

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [5, 10, 15, 20, 25, 30, 35])
@pytest.mark.parametrize("Do,D", [(64, 128), (2048, 2048)])
def test_f32_weight_gradient_of_a_few_rows(N, Do, D):
    """Runs of 8 k of a single K tile: 1 to 4 of them, and two tiles (35); 64 x
    64 and 128 x 128 block tiles."""
    tiles.test_layer_products_within_the_rounding_bound(1, N, Do, D)


@pytest.mark.parametrize("B,Do,D", [
    (5, 64, 64),       # one partial 128 x 128 tile, one K tile
    (130, 128, 192),   # the second row and column tiles partial, two K tiles
    (645, 128, 1024),  # 3 x 4 tiles of 256 x 256 would be: 6 x 8 of 128 x 128
    (645, 192, 1024),  # three K tiles: past the rule
    (4100, 128, 1024),  # 17 x 4 = 68 tiles of 256 x 256: past it
])
def test_bf16_short_k_within_the_rounding_bound(B, Do, D):
    tiles.test_tall_bf16_tiles_within_the_rounding_bound(B, Do, D)
