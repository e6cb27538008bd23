"""GPU: the fp32 matrix products take subnormal operands and give subnormal
results (nothing is flushed to zero), through the pre-LSTM layer.  Bound: K fp32
products and sums, each rounded once, to a multiple of 2^-149 at the smallest."""
import pytest
import torch

from paper_1912_06680_amd import o5
from tests.gpu_util import banner, need_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("so,sw", [(1e-40, 1e10), (1e-25, 1e-15)], ids=["operands", "results"])
@pytest.mark.parametrize("N,D", [(130, 128), (2050, 2048)])
def test_subnormal_values_are_kept(so, sw, N, D):
    need_gpu()
    banner(f"subnormal {so} x {sw} N={N} D={D}")
    Do = 64
    g = torch.Generator(device="cuda")
    g.manual_seed(N)
    o = torch.randn((N, Do), generator=g, device="cuda") * so
    W = torch.randn((D, Do), generator=g, device="cuda") * sw
    y, x = torch.empty((N, D), device="cuda"), torch.empty((N, D), device="cuda")
    o5.o5_prelstm_fwd(o5.O5_F32, 1, N, Do, D, o, W, torch.zeros(D, device="cuda"), y, x)
    ref = torch.relu(o.double() @ W.double().t())
    terms = o.double().abs() @ W.double().abs().t()
    bound = (Do + 2) * (2.0 ** -24 * terms + 2.0 ** -149)
    assert float(ref.max()) > 0 and float(((y.double() - ref).abs() / bound).max()) <= 1.0
