"""Vocabulary statistics of 129 - 256 rows of d_model <= 512: one row tile of 256, tiles of 128 columns, at most 256 of them; for a verify pass,
and the arg-max alone for a drafter's."""
import pytest

import test_gpu_vocab_tail as tail

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,B,k,V", [
    (512, 43, 2, 32768),      # 129 rows, 256 tiles: the most
    (512, 64, 3, 1003),       # 256 rows, the last tile cut
    (512, 51, 4, 32641),      # 255 rows, one column in the last tile
    (64, 43, 2, 130),         # K = 64: one stage
    (128, 32, 7, 300),        # K = 128: two, of a ring of three
])
def test_tall_tiles(d, B, k, V):
    tail.test_tail_against_oracle(d, B, k, V, {})


@pytest.mark.parametrize("d,B,k,V", [
    (512, 43, 3, 32768),      # 129 rows, 256 tiles: the most
    (512, 24, 10, 1003),      # 240, the last tile cut
    (512, 64, 4, 32641),      # 256, one column in the last tile
    (64, 43, 3, 130),
    (128, 51, 5, 300),
])
def test_tall_tiles_of_a_drafter(d, B, k, V):
    tail.test_drafter_tail(d, B, k, V)
