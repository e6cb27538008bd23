"""GPU: a reset cuts the carried state and its gradient off whatever they hold.
With infinities and NaN in what the reset masks, every kernel path gives the
outputs that finite values there give, bit for bit."""
import pytest
import torch

from paper_1912_06680_amd import o5
from tests.gpu_util import banner, need_gpu, workspace

pytestmark = pytest.mark.gpu

SHAPES = [
    (False, 17, 64, 128),    # one launch per step, forward and backward
    (False, 17, 64, 512),    # backward: product and cell
    (False, 4097, 64, 512),  # forward: product and cell
    (True, 17, 64, 128),     # one launch per step
    (True, 320, 64, 1024),   # backward: product and cell
    (True, 576, 64, 1024),   # forward: product and cell
    (True, 4096, 64, 1024),  # forward: the cell in the product's epilogue
]


def _case(bf16, B, D, H):
    T, et, dt = 2, torch.bfloat16 if bf16 else torch.float32, o5.O5_BF16 if bf16 else o5.O5_F32
    g = torch.Generator(device="cuda")
    g.manual_seed(B + H)

    def rnd(*s, std=1.0):
        return torch.randn(s, generator=g, device="cuda") * std

    x, Wx, Wh = rnd(T, B, D).to(et), rnd(4 * H, D, std=D ** -0.5).to(et), rnd(4 * H, H, std=0.5 * H ** -0.5).to(et)
    b, h0, c0, dh = rnd(4 * H, std=0.1), rnd(B, H, std=0.3), rnd(B, H, std=0.3), rnd(T, B, H)
    reset = torch.zeros((T, B), dtype=torch.uint8, device="cuda")
    reset[0, ::3] = 1
    reset[1, 1::3] = 1
    ws = workspace(max(o5.o5_lstm_fwd_workspace_bytes(dt, T, B, D, H), o5.o5_lstm_bptt_workspace_bytes(dt, T, B, D, H)))

    def run(h0, c0, dh):
        h, c = torch.empty((T, B, H), dtype=et, device="cuda"), torch.empty((T, B, H), device="cuda")
        gates = torch.empty((T, B, 4 * H), dtype=et, device="cuda")
        out = dict(dWx=torch.empty((4 * H, D), device="cuda"), dWh=torch.empty((4 * H, H), device="cuda"),
                   db=torch.empty(4 * H, device="cuda"), dx=torch.empty((T, B, D), dtype=et, device="cuda"))
        o5.o5_lstm_fwd(dt, T, B, D, H, x, Wx, Wh, b, h0, c0, reset, h, c, gates, ws)
        o5.o5_lstm_bptt(dt, T, B, D, H, x, Wx, Wh, h0, c0, reset, h, c, gates, dh, None, None, out["dWx"], out["dWh"],
                        out["db"], out["dx"], ws)
        return dict(h=h, c=c, gates=gates, **out)

    return run, h0, c0, dh, reset


@pytest.mark.parametrize("bf16,B,D,H", SHAPES)
def test_reset_masks_a_non_finite_stored_state(bf16, B, D, H):
    need_gpu()
    banner(f"reset over a non-finite state bf16={bf16} B={B} H={H}")
    run, h0, c0, dh, reset = _case(bf16, B, D, H)
    ref = run(h0, c0, dh)
    masked = reset[0] != 0
    h1, c1 = h0.clone(), c0.clone()
    h1[masked] = float("inf")
    c1[masked] = float("nan")
    c1[masked, ::2] = -float("inf")
    got = run(h1, c1, dh)
    for k in ref:
        assert torch.isfinite(ref[k].float()).all(), k
        assert torch.equal(got[k], ref[k]), k


@pytest.mark.parametrize("bf16,B,D,H", SHAPES)
def test_reset_masks_a_non_finite_later_gradient(bf16, B, D, H):
    need_gpu()
    banner(f"reset over a non-finite gradient bf16={bf16} B={B} H={H}")
    run, h0, c0, dh, reset = _case(bf16, B, D, H)
    ref = run(h0, c0, dh)
    bad = dh.clone()
    bad[1, reset[1] != 0] = float("inf")
    got = run(h0, c0, bad)
    assert torch.isfinite(ref["dx"][0].float()).all()
    assert torch.equal(got["dx"][0], ref["dx"][0])
