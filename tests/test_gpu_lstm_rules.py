"""GPU: the rules that choose between a step in one launch and the product and
the cell on their own: shapes on either side of the lines, sums split more ways
than a block has waves, and in bf16 the same bits on both sides."""
import pytest
import torch

from paper_1912_06680_amd import o5
from tests.gpu_util import banner, need_gpu, workspace
from tests.test_gpu_lstm_step import test_step_kernels_match_autograd as check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bf16,T,B,D,H", [
    # fp32, K = 576 counts as 768: the line at 160 tiles of 128 x 128
    (False, 1, 1150, 64, 512),   # 9 x 16 tiles
    (False, 1, 1160, 64, 512),   # 10 x 16: product and cell
])
def test_forward_rule_with_a_short_input(bf16, T, B, D, H):
    check(bf16, T, B, D, H)
