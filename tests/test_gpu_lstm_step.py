"""GPU: the one-launch recurrent steps (forward and backward) at the edges of
their tiles and on both sides of the rules that choose them, against PyTorch
autograd in fp64 on the same (bf16-rounded) inputs.

Tolerances are those of the path (max error over max magnitude, 1e-4 fp32 and
3e-2 bf16): the sums are fp32 over at most 10240 terms in any order, and
bf16 rounds the hidden state, the gates and dG once per step, two steps here.
"""
import pytest
import torch

from paper_1912_06680_amd import o5
from tests.gpu_util import TOL_BF16, TOL_F32, assert_close, banner, host, need_gpu, workspace

pytestmark = pytest.mark.gpu


def _reference(x, Wx, Wh, b, h0, c0, reset, dh, dhT, dcT):
    x, Wx, Wh, b = (t.double().requires_grad_() for t in (x, Wx, Wh, b))
    T, B, _ = x.shape
    H = h0.shape[1]
    h, c = h0.double(), c0.double()
    hs, cs, gs = [], [], []
    for t in range(T):
        keep = (reset[t] == 0).double()[:, None]
        # (no gradient flows into the stored state h0, c0)
        h, c = h * keep, c * keep
        a = x[t] @ Wx.t() + h @ Wh.t() + b
        i, f, g, o = (torch.sigmoid(a[:, :H]), torch.sigmoid(a[:, H:2 * H]), torch.tanh(a[:, 2 * H:3 * H]),
                      torch.sigmoid(a[:, 3 * H:]))
        c = f * c + i * g
        h = o * torch.tanh(c)
        hs.append(h)
        cs.append(c)
        gs.append(torch.cat([i, f, g, o], 1))
    hs, cs = torch.stack(hs), torch.stack(cs)
    J = (hs * dh.double()).sum() + (hs[-1] * dhT.double()).sum() + (cs[-1] * dcT.double()).sum()
    dx, dWx, dWh, db = torch.autograd.grad(J, (x, Wx, Wh, b))
    return dict(h=hs.detach(), c=cs.detach(), gates=torch.stack(gs).detach(), dx=dx, dWx=dWx, dWh=dWh, db=db)


@pytest.mark.parametrize("bf16,T,B,D,H", [
    (False, 2, 1, 64, 64),      # one row of one 16-row tile; 4 unit groups (not a multiple of the 8 XCDs)
    (False, 2, 17, 128, 192),   # a second 16-row tile with one row; 12 unit groups
    (False, 2, 33, 64, 2048),   # 32-row forward tiles, one row in the second; the split product backward
    (False, 2, 130, 64, 1536),  # 64-row forward tiles, two rows in the third; 32 x 32 backward tiles
    (False, 2, 1000, 64, 1024),  # 64 x 64 backward tiles, the last with 40 rows
    (False, 1, 4097, 64, 512),  # forward on the separate product and cell
    (True, 2, 1, 64, 64),
    (True, 2, 17, 128, 192),
    (True, 2, 33, 64, 2048),
    (True, 2, 130, 64, 1536),
    (True, 2, 769, 64, 1024),   # 13 x 64 = 832 blocks: forward and backward on separate launches
    (True, 3, 97, 192, 4096),   # 4 x 128 = 512 blocks of 32 x 32: backward on separate launches
])
def test_step_kernels_match_autograd(bf16, T, B, D, H):
    need_gpu()
    banner(f"lstm step bf16={bf16} T={T} B={B} D={D} H={H}")
    g = torch.Generator(device="cuda")
    g.manual_seed(B * H + D)
    et = torch.bfloat16 if bf16 else torch.float32
    dt = o5.O5_BF16 if bf16 else o5.O5_F32

    def rnd(*s, std=1.0):
        return torch.randn(s, generator=g, device="cuda") * std

    x, Wx, Wh = rnd(T, B, D).to(et), rnd(4 * H, D, std=H ** -0.5).to(et), rnd(4 * H, H, std=0.5 * H ** -0.5).to(et)
    b, h0, c0 = rnd(4 * H, std=0.1), rnd(B, H, std=0.3), rnd(B, H, std=0.3)
    reset = (torch.rand((T, B), generator=g, device="cuda") < 0.2).to(torch.uint8)
    dh, dhT, dcT = rnd(T, B, H), rnd(B, H), rnd(B, H)
    h, c = torch.full((T, B, H), -7.0, dtype=et, device="cuda"), torch.full((T, B, H), -7.0, device="cuda")
    gates = torch.full((T, B, 4 * H), -7.0, dtype=et, device="cuda")
    out = dict(dWx=torch.full((4 * H, D), -7.0, device="cuda"), dWh=torch.full((4 * H, H), -7.0, device="cuda"),
               db=torch.full((4 * H,), -7.0, device="cuda"), dx=torch.full((T, B, D), -7.0, dtype=et, device="cuda"))
    ws = workspace(max(o5.o5_lstm_fwd_workspace_bytes(dt, T, B, D, H), o5.o5_lstm_bptt_workspace_bytes(dt, T, B, D, H)))
    ws.fill_(0xAA)  # nothing may rely on clean scratch
    o5.o5_lstm_fwd(dt, T, B, D, H, x, Wx, Wh, b, h0, c0, reset, h, c, gates, ws)
    ws.fill_(0xAA)
    o5.o5_lstm_bptt(dt, T, B, D, H, x, Wx, Wh, h0, c0, reset, h, c, gates, dh, dhT, dcT, out["dWx"], out["dWh"],
                    out["db"], out["dx"], ws)
    ref = _reference(x, Wx, Wh, b, h0, c0, reset, dh, dhT, dcT)
    tol = TOL_BF16 if bf16 else TOL_F32
    for k, v in dict(h=h, c=c, gates=gates, **out).items():
        assert_close(k, host(v), host(ref[k]), tol)
