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


@pytest.mark.parametrize("T,B,D,H", [
    (2, 128, 4096, 1024),  # eight partial sums: each wave's second run
    (2, 60, 4096, 1024),
    (2, 128, 4096, 512),   # eight of 9 pieces: both runs of a wave odd
    (2, 33, 1152, 64),     # two sums of 10 and 9 pieces: an odd run is padded by a piece of zeros
    (2, 33, 2112, 64),     # four sums of 9, 9, 9 and 7 pieces
    (2, 33, 3008, 64),     # six sums of 8: some waves have a second run, others none
])
def test_forward_step_with_more_sums_than_waves(T, B, D, H):
    check(True, T, B, D, H)


def _bits(T, D, H, small, large, backward):
    """Outputs of `large` samples, and of their first `small` alone."""
    need_gpu()
    banner(f"bits on both paths B={small} and {large} D={D} H={H} backward={backward}")
    et, dt, ld = torch.bfloat16, o5.O5_BF16, 256
    g = torch.Generator(device="cuda")
    g.manual_seed(H + large)

    def rnd(*s, std=1.0):
        return torch.randn(s, generator=g, device="cuda") * std

    x, Wx, Wh = rnd(T, large, D).to(et), rnd(4 * H, D, std=D ** -0.5).to(et), rnd(4 * H, H, std=0.5 * H ** -0.5).to(et)
    b, h0, c0 = rnd(4 * H, std=0.1), rnd(large, H, std=0.3), rnd(large, H, std=0.3)
    P, W = rnd(T, large, ld, std=0.1).to(et), rnd(H, ld, std=0.1).to(et)
    dh = rnd(T, large, H)
    reset = (torch.rand((T, large), generator=g, device="cuda") < 0.1).to(torch.uint8)
    out = []
    for B in (large, small):
        xs, rs, Ps, dhs = (v[:, :B].contiguous() for v in (x, reset, P, dh))
        hs, cs = h0[:B].contiguous(), c0[:B].contiguous()
        h, c = torch.empty((T, B, H), dtype=et, device="cuda"), torch.empty((T, B, H), device="cuda")
        gates = torch.empty((T, B, 4 * H), dtype=et, device="cuda")
        o5.o5_lstm_fwd(dt, T, B, D, H, xs, Wx, Wh, b, hs, cs, rs, h, c, gates,
                       workspace(o5.o5_lstm_fwd_workspace_bytes(dt, T, B, D, H)))
        got = dict(h=h, c=c, gates=gates)
        if backward:
            dx = torch.empty((T, B, D), dtype=et, device="cuda")
            grads = (torch.empty((4 * H, D), device="cuda"), torch.empty((4 * H, H), device="cuda"),
                     torch.empty(4 * H, device="cuda"), dx)
            ws = workspace(o5.o5_lstm_bptt_workspace_bytes(dt, T, B, D, H))
            if backward == "factored":
                o5.o5_lstm_bptt_factored(dt, T, B, D, H, xs, Wx, Wh, hs, cs, rs, h, c, gates, Ps.view(T * B, ld), W, ld,
                                         None, None, *grads, ws)
            else:
                o5.o5_lstm_bptt(dt, T, B, D, H, xs, Wx, Wh, hs, cs, rs, h, c, gates, dhs, None, None, *grads, ws)
            got["dx"] = dx
        out.append(got)
    for k in out[0]:
        assert torch.equal(out[0][k][:, :small], out[1][k]), k


def test_forward_bits_do_not_depend_on_the_path():
    """512 samples take one launch per step (512 blocks), 576 the product, split
    in two for both batches, and the cell."""
    _bits(3, 64, 1024, 512, 576, None)


@pytest.mark.parametrize("backward", ["factored", "plain"])
def test_backward_bits_do_not_depend_on_the_path(backward):
    """256 samples take one launch per backward step (256 blocks), 320 the
    product, split in eight for both batches, and the cell; dx holds dG's bits."""
    _bits(3, 64, 1024, 256, 320, backward)
