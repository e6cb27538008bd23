"""GPU parity: o5_segments_to_samples with eight elements per thread and tile
(calls of 524,288 elements and more), bit for bit against the oracle."""
import pytest

from tests.test_gpu_cut_tiles import test_segments_to_samples_tiles as check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,S,T", [
    (256, 2113, 4),   # 64 samples a segment: two tiles of 32 x 64, the fullest layout; the last tile one segment wide
    (70, 8193, 2),    # 35: a second tile of three
    (256, 2050, 16),  # 16 x 128, the last tile two segments wide
    (99, 8191, 33),   # 3 samples a segment, no power of two; the last tile one short
    (17, 30841, 17),  # one sample a segment: 1 x 2048
])
def test_segments_to_samples_large_tiles(L, S, T):
    assert L * S >= 256 * 2048
    check(L, S, T)
