"""The end of a verify pass: the last LayerNorm and the drafts' logits in one launch (d_model 512 / 1024, 16 rows a block), and the
vocabulary tiles by which they are chosen: 128 x 128 with a deep ring where every block has a CU of its own, with a short one where
not, 256 x 256 from one to a CU, several of them to a block beyond (K a multiple of 128)."""
import numpy as np
import pytest

import cases
import gpu_harness as gh
import specdec_oracle as orc
import test_gpu_parity_extra as extra
from paper_2203_16487_amd import binding as sd
from paper_2203_16487_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,B,k,V,opts", [
    (512, 11, 2, 1003, {}),                                       # 33 rows: a last block of one row
    (512, 4, 11, 777, {}),                                        # 48 rows: whole blocks
    (512, 11, 2, 33000, {}),                                      # 258 tiles: the short ring
    (512, 23, 5, 32800, {}),                                      # 138 rows, 514 tiles of 128 x 128: the short ring
    (1024, 11, 2, 32768, {}),                                     # 256 tiles: the deep ring's most
    (1024, 9, 6, 1003, {}),                                       # 63 rows
    (1024, 13, 4, 300, {sd.SPECDEC_OPT_WIDE_VOCAB_TILES: 1}),     # 65 rows, 256 x 256 tiles
    (512, 43, 5, 32768, {}),                                      # 258 rows, 256 tiles of 256 x 256: the fewest by themselves
    (512, 65, 7, 32100, {}),                                      # 520 rows, 378 tiles of 256 x 256: the second round in halves, the last of them cut away
    (256, 65, 7, 33000, {}),                                      # K = 256, the shortest of them
    (512, 65, 7, 32896, {}),                                      # 387 tiles, a half tile of rows and columns at the end
    (512, 127, 6, 25600, {}),                                     # 400 tiles: more than half a round, whole tiles
    (192, 65, 7, 32100, {}),                                      # K = 192: a block a tile
    (128, 11, 2, 1003, {}),                                       # another width: two launches
])
def test_tail_against_oracle(d, B, k, V, opts):
    desc = synth.ModelDesc(0, 1, d, d // 64, 2 * d, V, 16, 64).resolved()
    case = cases.make_verify_case(desc, seed=d + B + k, B=B, k=k, S=9, beta=3, tau=1.0, len_lo=0, len_hi=12, drafts="greedy",
                                  ragged_src=True)
    cases.run_oracle(case)
    drafts = case.drafts.copy()
    ses = gh.open_verifier(case, options=opts, fill=0xFF)
    out = gh.gpu_verify(ses, case, drafts)
    bare = gh.gpu_verify(ses, case, drafts, want_logits=False)
    ses.close()
    err = float(np.abs(out["logits"] - case.logits).max())
    assert err <= max(2e-2, 0.04 * float(case.logits.std())), err
    assert not cases.compare_decisions(case, out["accept"], out["next"])[2]
    z, st = out["logits"], out["stats"]
    zd = np.take_along_axis(z[:, :k], drafts[:, :, None].astype(np.int64), axis=2)[..., 0]
    assert np.array_equal(st[:, :k, 3], zd)                                        # the drafts' logits, to the last bit
    assert np.array_equal(st[:, :k, 4], (z[:, :k] > zd[..., None]).sum(-1).astype(np.float32))
    assert np.array_equal(st[..., 0], z.max(-1)) and np.array_equal(st[..., 1].astype(np.int64), z.argmax(-1))
    assert np.array_equal(bare["stats"], st)
    assert np.array_equal(bare["accept"], out["accept"]) and np.array_equal(bare["next"], out["next"])


@pytest.mark.parametrize("d,B,k,V", [
    (512, 65, 8, 32100),      # 520 rows, 378 tiles of 256 x 256: the second round in halves, the last of them cut away
    (256, 65, 8, 32896),      # 387, a half tile of rows and columns at the end
    (512, 26, 10, 32768),     # 260 rows, 256 tiles
])
def test_drafter_tail(d, B, k, V):
    """A drafter's pass: every row's arg-max with the logits asked for and (another kernel) without, two sequences against the oracle."""
    desc = synth.ModelDesc(1, 1, d, d // 64, 2 * d, V, 16, 64).resolved()
    bits = synth.make_weights(desc, d + V, tag="drafter")
    extra.drafter_pass_case(desc, bits, orc.Model(desc, synth.weights_f32(bits)), B=B, S_max=9, k=k, lens=synth.random_lengths(d, "len", B, 0, 12),
                            seed=d + B, prefill=True, sample=(0, B - 1), max_tgt=40)
