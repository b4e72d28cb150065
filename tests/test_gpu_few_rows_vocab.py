"""Vocabulary statistics of passes of at most 32 rows: one row tile and two with their remainders, a tile of 64 columns to a block and two
(beyond 256 of them), a last block of one tile and one that the vocabulary's end cuts, bf16 weights and codes, d = 128, 512 and
1024 (half of the bf16 weights requested behind the LayerNorm)."""
import numpy as np
import pytest

import cases
import gpu_harness as gh
from paper_2203_16487_amd import binding as sd
from paper_2203_16487_amd import synth

pytestmark = pytest.mark.gpu

FFN = {128: 256, 512: 2048, 1024: 4096}


@pytest.mark.parametrize("d,B,k,V,fp8", [
    (128, 1, 1, 130, False),        # 2 rows; 3 tiles
    (128, 2, 15, 1003, True),       # 32 rows
    (512, 1, 15, 1003, False),      # 16 rows: one row tile, whole
    (512, 1, 16, 1050, False),      # 17; 17 tiles
    (512, 3, 4, 704, True),         # 15
    (512, 4, 6, 705, True),         # 28
    (1024, 1, 1, 1003, False),
    (1024, 2, 15, 1050, False),     # 32
    (1024, 1, 25, 32768, True),     # 26, a block to a CU
    (1024, 1, 5, 200, True),
    (128, 2, 15, 16384, True),      # 256 tiles: the most of which a block takes one
    (512, 1, 15, 16384, False),
    (512, 1, 16, 16385, False),     # 257: the last block has one, of one column
    (128, 1, 4, 16449, True),       # 258, the last of one column
    (512, 3, 4, 16500, True),
    (1024, 1, 15, 16449, False),
    (1024, 2, 15, 16385, False),
])
def test_few_rows_vocab(d, B, k, V, fp8):
    desc = synth.ModelDesc(0, 1, d, d // 64, FFN[d], V, 16, 64).resolved()
    case = cases.make_verify_case(desc, seed=d + B + k, B=B, k=k, S=9, beta=3, tau=1.0, len_lo=0, len_hi=12, drafts="greedy", ragged_src=True,
                                  fp8=fp8)
    cases.run_oracle(case)
    ses = gh.open_verifier(case, options={sd.SPECDEC_OPT_FP8_WEIGHTS: int(fp8)}, fill=0xFF)
    out = gh.gpu_verify(ses, case)
    bare = gh.gpu_verify(ses, case, want_logits=False)
    ses.close()
    err = float(np.abs(out["logits"] - case.logits).max())
    assert err <= max(2e-2, 0.04 * float(case.logits.std())), err
    assert not cases.compare_decisions(case, out["accept"], out["next"])[2]
    z, st = out["logits"], out["stats"]
    zd = np.take_along_axis(z[:, :k], case.drafts[:, :, None].astype(np.int64), axis=2)[..., 0]
    assert np.array_equal(st[:, :k, 3], zd)                                        # the drafts' logits, to the last bit
    assert np.array_equal(st[:, :k, 4], (z[:, :k] > zd[..., None]).sum(-1).astype(np.float32))
    assert np.array_equal(st[..., 0], z.max(-1)) and np.array_equal(st[..., 1].astype(np.int64), z.argmax(-1))
    lse = np.log(np.exp(z.astype(np.float64) - z.max(-1, keepdims=True)).sum(-1)) + z.max(-1)
    assert np.abs(st[..., 2] - lse).max() <= 1e-4                                   # fp32 exponentials (2^-21) and sums of positive terms: 1e-5 at most, with a margin
    assert np.array_equal(bare["stats"], st)
