"""CPU: workspace queries hold what the chosen kernels read and no more."""
import pytest

from paper_1912_06680_amd import o5


def _up(n):
    return (n + 255) // 256 * 256


def _bptt_bf16_bytes(T, B, D, H, splits):
    """dG, dc, the recurrent product's partial sums, bf16 h0, the bias
    gradient's partial rows, dG^T, [x | h~]^T and W_h^T (time padded to 64)."""
    Bp = (B + 63) // 64 * 64
    ldt = T * Bp
    return (_up(T * B * 4 * H * 2) + _up(B * H * 4) + _up(splits * B * H * 4) + _up(B * H * 2)
            + _up(Bp // 32 * 4 * H * 4) + _up(4 * H * ldt * 2) + _up((D + H) * ldt * 2) + _up(4 * H * H * 2))


@pytest.mark.parametrize("T,B,D,H", [(16, 8, 4096, 4096), (1, 1, 65536, 64), (2, 256, 16384, 4096),
                                     (16, 2048, 4096, 4096), (16, 600, 4096, 4096), (3, 130, 1024, 64)])
def test_bptt_bf16_transposed_input_weights_need_no_room_of_their_own(T, B, D, H):
    got = o5.o5_lstm_bptt_workspace_bytes(o5.O5_BF16, T, B, D, H)
    assert 0 < got <= _bptt_bf16_bytes(T, B, D, H, 8)


@pytest.mark.parametrize("T,B,D,H", [(16, 60, 4096, 4096), (16, 256, 4096, 4096), (2, 1000, 64, 1024), (1, 1, 64, 64)])
def test_bptt_fp32_transposed_recurrent_weights_need_no_room(T, B, D, H):
    """dG, dc, the recurrent product's partial sums (at most 16), and the bias
    gradient's partial rows; W_h^T waits in the output dW_h."""
    Bp = (B + 63) // 64 * 64
    most = (_up(T * B * 4 * H * 4) + _up(B * H * 4) + _up(16 * B * H * 4) + _up(B * H * 4) + _up(Bp // 32 * 4 * H * 4))
    assert 0 < o5.o5_lstm_bptt_workspace_bytes(o5.O5_F32, T, B, D, H) <= most


@pytest.mark.parametrize("dt,N,H,heads,ku,d", [
    (o5.O5_BF16, 9600, 4096, (30, 189, 32, 4), 1, 128),
    (o5.O5_BF16, 600, 1024, (30, 40, 4), 1, 64),
    (o5.O5_F32, 9600, 512, (400, 30), 0, 64),
])
def test_unit_head_adds_what_the_one_pass_kernel_reads(dt, N, H, heads, ku, d):
    """A unit head whose rows the one-pass kernel takes adds the query's
    partial sums, the d column sums, in bf16 the pair's and the weights'
    columns and their partial sums, in fp32 dq and the partial sums of dWq;
    no logits or gradients per unit, no second copy of dq."""
    plain = o5.o5_ppo_loss_grad_workspace_bytes(dt, N, H, heads)
    got = o5.o5_ppo_loss_grad_workspace_bytes(dt, N, H, heads, o5.unit_head(ku, d, None, None, None))
    dp, A1 = (d + 63) // 64 * 64, sum(heads) + 1
    A1p = (A1 + 63) // 64 * 64
    blocks = min(N, 1024)
    more = 8 * N * d * 4 + 4 * (blocks + 1) * (A1 + 8 + d) + 4096
    if dt == o5.O5_BF16:
        tiles = -(-2 * (A1p + dp) // 256) * -(-H // 256)
        splits = max(1, min(256 // tiles, -(-N // 32) // 8))
        more += N * 2 * dp * 2 + H * 2 * dp * 2 + splits * 2 * (A1p + dp) * H * 4
    else:
        more += N * d * 4 + 16 * d * H * 4
    assert plain < got <= plain + more
