"""The projections' larger tiles (128 x 128 with a ring of four, 256 x 128, 128 x 128 two to a CU, 256 x 256, one or several of these
to a block), each where the rule first and last takes it: widths that end inside a tile, rows that end inside one, rows that the call only bounds; outputs, sums
with their statistics, and keys / values appended to the cache."""
import numpy as np
import pytest
import torch

import cases
import gpu_harness as gh
from paper_2203_16487_amd import binding as sd
from paper_2203_16487_amd import synth
import specdec_oracle as orc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,F,B,S,lo", [
    (192, 2112, 16, 63, 63),      # 1008 rows: 136 tiles of 128 x 128 (FFN1)
    (192, 2112, 131, 64, 40),     # bound 8384 rows: sums of 132, QKV of 330, FFN1 of 1122
    (192, 2112, 257, 65, 1),      # bound 16705 rows: sums of 262
    (512, 2048, 64, 129, 129),    # 8256 rows: sums of 260
    (512, 2048, 128, 128, 90),    # bound 16384 rows: sums of 512 (256 x 128, one to a CU), FFN1 of 256 x 256, two or three to a block
    (512, 2112, 129, 128, 100),   # FFN1: the last tile of a row 64 columns wide (half of it empty)
    (256, 2048, 256, 128, 128),   # K = 256, the shortest of them: four whole tiles to a block
    (512, 2048, 129, 128, 1),     # half the rows that the grid is sized for: 264 tiles, the last ones in halves
    (1024, 4096, 20, 450, 450),   # 9000 rows, K = 1024: QKV (22 of an XCD's round left: whole tiles) and FFN1 (8: halves)
])
def test_encoder_tiles(d, F, B, S, lo):
    desc = synth.ModelDesc(1, 1, d, d // 64, F, 1000, S, 16).resolved()
    bits = synth.make_weights(desc, B, std=0.04)
    model = orc.Model(desc, synth.weights_f32(bits))
    src = synth.random_tokens(B, "src", (B, S), desc)
    lens = np.random.default_rng(B).integers(lo, S + 1, B).astype(np.int32)
    ses = sd.Session(B, 4, S, 16, fill=0xFF)
    ses.bind_model(sd.SPECDEC_VERIFIER, desc, ses.upload_weights(bits))
    sd.specdec_begin(ses.ctx, B, 8)
    sd.specdec_encode(ses.ctx, ses.i32(src), ses.i32(lens))
    mem = torch.zeros((B, S, d), dtype=torch.bfloat16, device=ses.device)
    sd.specdec_get_memory(ses.ctx, sd.SPECDEC_VERIFIER, mem)
    torch.cuda.synchronize()
    got = mem.float().cpu().numpy()
    ses.close()
    for b in list(range(0, B, 9)) + [B - 1]:
        n = int(lens[b])
        err = float(np.abs(got[b, :n] - orc.encode(model, [int(t) for t in src[b, :n]])).max())
        assert err <= 3e-2, (b, n, err)


@pytest.mark.parametrize("B,k", [
    (128, 10),      # 1408 rows: 132 tiles of 128 x 128 (QKV), 176 (FFN1)
    (125, 22),      # 2875 rows, the last tile cut: 276 and 368 tiles
])
def test_decoder_tiles(B, k):
    desc = synth.ModelDesc(0, 1, 512, 8, 2048, 1003, 12, 64).resolved()
    case = cases.make_verify_case(desc, seed=B, B=B, S=12, k=k, beta=3, tau=1.0, len_lo=0, len_hi=9, drafts="random", ragged_src=True)
    cases.run_oracle(case)
    ses = gh.open_verifier(case, fill=0xFF)
    out = gh.gpu_verify(ses, case)
    K, V = gh.gpu_cache(ses, case, case.L_max + k + 1)
    ses.close()
    err = float(np.abs(out["logits"] - case.logits).max())
    assert err <= max(2e-2, 0.04 * float(case.logits.std())), err
    assert not cases.compare_decisions(case, out["accept"], out["next"])[2]
    for b, st in enumerate(case.states):
        j = int(case.lens[b])
        assert np.abs(K[0, b, j:j + k + 1] - st.K[0][j:j + k + 1]).max() <= 3e-2, b
        assert np.abs(V[0, b, j:j + k + 1] - st.V[0][j:j + k + 1]).max() <= 3e-2, b


def test_prefill_tiles():
    """Some 6300 rows of d = 1024: queries, keys and values of 300 tiles of 256 x 256, six left of every XCD's round, in halves."""
    desc = synth.ModelDesc(0, 1, 1024, 16, 4096, 1000, 16, 64).resolved()
    case = cases.make_verify_case(desc, seed=3, B=32, S=7, k=4, beta=3, tau=1.0, len_lo=190, len_hi=205, drafts="random", ragged_src=True,
                                  std=0.015)
    L = case.L_max
    K, V = cases.oracle_flat_cache(case, L)
    ses = gh.open_verifier(case, max_tgt=216, fill=0xFF)
    sd.specdec_set_stream(ses.ctx, ses.i32(case.tokens), ses.i32(case.lens))   # nothing counts as cached any more
    zeros = torch.zeros((1, 32, L, 1024), dtype=torch.bfloat16, device=ses.device)
    sd.specdec_load_cache(ses.ctx, sd.SPECDEC_VERIFIER, zeros, zeros, ses.i32(np.zeros(32, np.int32)))
    sd.specdec_set_stream(ses.ctx, ses.i32(case.tokens), ses.i32(case.lens))
    sd.specdec_prefill(ses.ctx, sd.SPECDEC_VERIFIER)
    gk, gv = gh.gpu_cache(ses, case, L)
    ses.close()
    for b in range(32):
        j = int(case.lens[b])
        assert np.abs(gk[:, b, :j] - K[:, b, :j]).max() <= 3e-2, b
        assert np.abs(gv[:, b, :j] - V[:, b, :j]).max() <= 3e-2, b
