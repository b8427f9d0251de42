"""Decode attention of 64 columns at both ends of the lengths that eight waves take in one step."""
import pytest
from test_gpu_decode_attention import test_rows_of_every_length_in_blocks as _check

pytestmark = pytest.mark.gpu


# bounds of 128 and 257 keys beside 129 and 256; rows that leave waves without keys, and whose last key is a wave's first or last
@pytest.mark.parametrize("H,KVH", [(4, 4), (8, 2), (8, 1)])
@pytest.mark.parametrize("slots", [(0, 31, 127), (5, 96, 128), (0, 33, 129, 159, 160, 191, 224, 255), (0, 200, 256)])
def test_rows_around_one_step(H, KVH, slots):
    _check(64, H, KVH, slots)
