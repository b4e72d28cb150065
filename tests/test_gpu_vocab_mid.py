"""Vocabulary statistics of 257 - 384 rows on tiles of 192 x 256 (two row tiles, one round of them), of 513 - 640 behind tiles of 256 x 128, and of more rows on tiles of 256 x 256 where those of 128 x
128 would be one round and some of a second; for a verify pass, and the arg-max alone for a drafter's."""
import pytest

import test_gpu_vocab_tail as tail
from paper_2203_16487_amd import binding as sd

pytestmark = pytest.mark.gpu
WIDE = {sd.SPECDEC_OPT_WIDE_VOCAB_TILES: 1}


@pytest.mark.parametrize("d,B,k,V,opts", [
    (512, 43, 5, 21761, {}),      # 258 rows: 66 in the second row tile; 513 tiles of 128 x 128, the fewest; one column in the last tile
    (512, 48, 7, 32768, {}),      # 384 rows, the most; 128 column tiles, the most
    (1024, 32, 10, 30000, {}),    # 352
    (512, 65, 4, 21760, {}),      # 325, 510: 128 x 128
    (64, 43, 5, 300, WIDE),       # K = 64: one stage
    (192, 48, 7, 513, WIDE),      # K = 192: three, of a ring of two; the last tile one column wide
    (512, 55, 6, 16500, {}),      # 385 rows, 516 of 128 x 128: 256 x 256, 130 of them
    (512, 46, 10, 28545, {}),     # 506 rows, 896: the most
    (256, 46, 10, 28673, {}),     # 900: 128 x 128
    (512, 57, 8, 21761, {}),      # 513 rows: 65 in the last row tile; the fewest column tiles, the last of one column
    (192, 64, 9, 32500, {}),      # 640, the most; the last tile of 256 x 128 cut
    (1024, 48, 10, 30000, {}),    # 528
    (512, 64, 9, 21760, {}),      # 256 x 256
])
def test_tiles(d, B, k, V, opts):
    tail.test_tail_against_oracle(d, B, k, V, opts)


@pytest.mark.parametrize("d,B,k,V", [
    (512, 43, 6, 21761),          # 258 rows
    (512, 32, 10, 32003),         # 320
    (512, 48, 8, 32768),          # 384
    (512, 40, 10, 20000),         # 400: 256 x 256
    (512, 64, 10, 32768),         # 640
    (512, 57, 9, 32003),          # 513
])
def test_tiles_of_a_drafter(d, B, k, V):
    tail.test_drafter_tail(d, B, k, V)
