"""GPU parity: the loss with a unit-selection head at the edges of its one-pass
row kernel (chunks of a row per thread, widths, columns per thread, rows
beyond one grid) and of the two-pass kernels that longer rows take, against
the fp64 oracle."""
import pytest

import tests.test_gpu_unit_head as head

pytestmark = pytest.mark.gpu

# a row of nk units is nk d / 8 chunks over 256 threads: 4, 12 and 16 chunks per
# thread are the one-pass variants, 17 is past them
EDGES = [
    (5, 64, (1, 2), 0, 8, True),            # a single chunk
    (3, 64, (2, 3), 1, 16, False),
    (1030, 64, (5, 7, 3), 1, 32, True),     # rows beyond one grid
    (70, 64, (64, 3), 0, 128, True),        # exactly 4
    (70, 64, (3, 65), 1, 128, False),       # 5
    (40, 64, (4, 193, 2), 1, 128, False),   # 13
    (40, 64, (30, 5), 0, 512, False),       # widest units
    (40, 64, (30, 5), 0, 256, True),
    (40, 64, (300, 20, 2), 1, 64, True),    # more than 256 columns
    (40, 64, (256, 2), 0, 128, True),       # exactly 16
    (40, 64, (256, 2), 0, 128, False),
    (40, 64, (257, 2), 0, 128, True),       # 17
    (40, 64, (2, 257), 1, 128, False),
]


@pytest.mark.parametrize("N,H,heads,ku,d,bf16", EDGES, ids=lambda v: str(v).replace(" ", ""))
def test_unit_head_row_lengths(N, H, heads, ku, d, bf16):
    name = f"edge nk={heads[ku]} d={d}"
    head.test_ppo_with_unit_head_matches_oracle(name, N, H, heads, ku, d, bf16, N % 2 == 0)
