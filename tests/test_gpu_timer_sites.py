"""The timed sites of an optimizer step whose LSTM steps run as one launch each:
the product's sites hold them, the cells' sites have no launches (so that no HBM
rate of a cell is formed from a launch that holds a product)."""
import pytest
import torch

import bench
from paper_1912_06680_amd import o5, synth
from paper_1912_06680_amd.step import PARAM_ORDER, PPOStep
from tests.gpu_util import banner, need_gpu


def test_recurrent_flop_counts_every_steps_products():
    B, T, H, ld = 8, 16, 128, 256
    plain = sum(2.0 * B * H * 4 * H for _ in range(T - 1))
    assert bench.recurrent_flop(B, T, H, 0) == plain
    assert bench.recurrent_flop(B, T, H, ld) == plain + sum(2.0 * B * H * ld for _ in range(T))


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_one_launch_steps_are_timed_as_products(dtype):
    need_gpu()
    banner(f"timer sites {dtype}")
    cfg = synth.scaled(synth.CONFIGS["tiny"], dtype=dtype)
    inp = synth.make_inputs(cfg, 0)
    st = PPOStep(cfg)
    st.load_params({k: inp[k] for k in PARAM_ORDER})
    st.load_x(inp["x"])
    st.load_rollout(inp["h0"], inp["c0"], inp["rewards"], inp["dones"], inp["rewards"][:1].repeat(cfg.L + 1, 0),
                    torch.zeros((st.N, len(cfg.head_sizes))).numpy(), torch.zeros(st.N).numpy())
    o5.o5_ktimer_enable(True)
    st.run()
    torch.cuda.synchronize()
    o5.o5_ktimer_enable(False)
    n = {name: o5.o5_ktimer_read(i)[1] for i, name in enumerate(o5.KTIMER_SITES)}
    assert n["lstm_fwd_gemm"] == cfg.T and n["lstm_dh_gemm"] == cfg.T
    assert n["lstm_fwd_cell"] == 0 and n["lstm_bwd_cell"] == 0
