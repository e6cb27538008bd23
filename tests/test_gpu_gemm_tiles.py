"""GPU: the matrix engines at the edges of their tiles, through the pre-LSTM
layer (fp32 forward: two K-contiguous operands; fp32 weight gradient: two
I-contiguous ones with a reduction length that is no multiple of the K tile;
bf16 forward: the tall tiles).

Bound: a sum of K fp32 products in any order is within (K + 2) 2^-24
sum_k |a_k b_k| of the exact one (each product and each add rounds once)."""
import pytest
import torch

from paper_1912_06680_amd import o5
from tests.gpu_util import banner, need_gpu, workspace

pytestmark = pytest.mark.gpu

U = 2.0 ** -24


def _within(name, got, ref, terms, k):
    err = (got.double() - ref).abs()
    bound = (k + 2) * U * terms + 1e-30
    worst = float((err / bound).max())
    print(f"    {name}: worst error / bound = {worst:.3f}", flush=True)
    assert worst <= 1.0, name


@pytest.mark.parametrize("T,B,Do,D", [
    (1, 5, 64, 64),        # one partial 64 x 64 tile, K = one run of two stages
    (13, 5, 64, 128),      # 65 rows: one row in the second tile; 65 = two stages + 1 in the weight gradient
    (1, 125, 192, 64),     # 125 rows, 3 stages of K beyond the first
    (1, 2050, 128, 2048),  # 17 x 16 tiles of 128 x 128, the last row tile with 2 rows
    (1, 2045, 2048, 2048),  # the weight gradient on 128 x 128 tiles over K = 2045
])
def test_layer_products_within_the_rounding_bound(T, B, Do, D):
    need_gpu()
    banner(f"f32 gemm T={T} B={B} Do={Do} D={D}")
    N = T * B
    g = torch.Generator(device="cuda")
    g.manual_seed(N + D)
    o = torch.randn((N, Do), generator=g, device="cuda")
    W = torch.randn((D, Do), generator=g, device="cuda")
    b = torch.zeros(D, device="cuda")
    y, x = torch.full((N, D), -7.0, device="cuda"), torch.empty((N, D), device="cuda")
    o5.o5_prelstm_fwd(o5.O5_F32, T, B, Do, D, o, W, b, y, x)
    pre = o.double() @ W.double().t()
    _within("y", y, torch.relu(pre), o.double().abs() @ W.double().abs().t(), Do)
    dx = torch.randn((N, D), generator=g, device="cuda")
    # equal positive outputs: every row is active and the first replica wins the pool
    ones = torch.ones((N, D), device="cuda")
    dW, db = torch.full((D, Do), -7.0, device="cuda"), torch.empty(D, device="cuda")
    ws = workspace(o5.o5_prelstm_bwd_workspace_bytes(o5.O5_F32, T, B, Do, D))
    o5.o5_prelstm_bwd(o5.O5_F32, T, B, Do, D, o, ones, dx, dW, db, ws)
    dpre = dx.clone().view(N // 5, 5, D)
    P = D // 4
    s = dpre[:, :, :P]
    tot = (((s[:, 0] + s[:, 1]) + s[:, 2]) + s[:, 3]) + s[:, 4]  # the pool's own fp32 sum
    dpre[:, :, :P] = 0
    dpre[:, 0, :P] = tot
    dpre = dpre.reshape(N, D).double()
    _within("dW", dW, dpre.t() @ o.double(), dpre.abs().t() @ o.double().abs(), N)


@pytest.mark.parametrize("B,Do,D", [
    (4805, 64, 4096),   # 16 x 16 tiles of 320 x 256, the last row tile with 5 rows; one K tile
    (5000, 192, 4096),  # the last row tile with 200 rows; three K tiles
    (5120, 320, 4032),  # whole row tiles, the last column tile with 192 columns
])
def test_tall_bf16_tiles_within_the_rounding_bound(B, Do, D):
    """320 x 256 tiles of the bf16 engine: products of bf16 values are exact
    in fp32, so the same bound holds for the sum (and y is stored in fp32)."""
    need_gpu()
    banner(f"bf16 tall tiles B={B} Do={Do} D={D}")
    g = torch.Generator(device="cuda")
    g.manual_seed(B)
    o = torch.randn((B, Do), generator=g, device="cuda").bfloat16()
    W = torch.randn((D, Do), generator=g, device="cuda").bfloat16()
    b = torch.randn(D, generator=g, device="cuda")
    y, x = torch.full((B, D), -7.0, device="cuda"), torch.empty((B, D), dtype=torch.bfloat16, device="cuda")
    o5.o5_prelstm_fwd(o5.O5_BF16, 1, B, Do, D, o, W, b, y, x)
    pre = o.double() @ W.double().t() + b.double()
    _within("y", y, torch.relu(pre), o.double().abs() @ W.double().abs().t() + b.double().abs(), Do + 1)
