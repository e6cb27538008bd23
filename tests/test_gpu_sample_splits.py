"""GPU parity: the sampler over the number of split sums of its logits product
(its row kernel has a variant for up to two and one for more, of which it loads
eight together), against the fp64 oracle."""
import pytest

import tests.test_gpu_ppo_sample as base

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bf16,B,H,heads", [
    (True, 60, 64, base.HEADS),          # one sum
    (True, 60, 512, base.HEADS),         # two
    (True, 60, 832, base.HEADS),         # three
    (True, 60, 2048, base.HEADS),        # eight
    (True, 7, 2048, base.MAX_LOGITS),    # eight, 16 columns per lane
    (False, 60, 128, base.HEADS),        # one
    (False, 60, 1152, base.HEADS),       # nine: one beyond the eight
    (False, 60, 2048, base.MAX_HEADS),   # sixteen
])
def test_policy_sample_split_sums(bf16, B, H, heads):
    base.test_policy_sample_matches_oracle(f"splits H={H}", B, H, bf16, H == 2048, heads)
