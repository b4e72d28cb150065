"""Attention of many queries per sequence (encoder passes): sources around the edges of the query and key tiles, one token
long and longer than a tile, against the oracle; and the tile kernel's choice of the keys it reads (buffers hold NaN)."""
import numpy as np
import pytest
import torch

from paper_2203_16487_amd import binding as sd
from paper_2203_16487_amd import synth
import specdec_oracle as orc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S,lens", [
    (33, (33, 1, 32, 31)),
    (65, (65, 64, 63, 2)),
    (129, (129, 128, 127, 66)),
    (300, (300, 257, 192, 8)),
])
def test_encoder_attention_edges(S, lens):
    desc = synth.ModelDesc(2, 1, 128, 2, 256, 1000, S, 16).resolved()
    bits = synth.make_weights(desc, S, std=0.06)
    model = orc.Model(desc, synth.weights_f32(bits))
    B = len(lens)
    src = synth.random_tokens(S, "src", (B, S), desc)
    ses = sd.Session(B, 4, S, 16, fill=0xFF)
    ses.bind_model(sd.SPECDEC_VERIFIER, desc, ses.upload_weights(bits))
    sd.specdec_begin(ses.ctx, B, 8)
    sd.specdec_encode(ses.ctx, ses.i32(src), ses.i32(np.asarray(lens, np.int32)))
    mem = torch.zeros((B, S, desc.d_model), dtype=torch.bfloat16, device=ses.device)
    sd.specdec_get_memory(ses.ctx, sd.SPECDEC_VERIFIER, mem)
    torch.cuda.synchronize()
    got = mem.float().cpu().numpy()
    for b, n in enumerate(lens):
        err = float(np.abs(got[b, :n] - orc.encode(model, [int(t) for t in src[b, :n]])).max())
        assert err <= 3e-2, (b, n, err)
    ses.close()


def test_encoder_attention_wide_scores():
    """Scores of standard deviation 6 (as exponents of 2): a row's maximum grows by less and by more than 8 from tile to tile."""
    S, lens = 300, (300, 251, 130, 65)
    desc = synth.ModelDesc(1, 1, 128, 2, 256, 1000, S, 16).resolved()
    bits = synth.make_weights(desc, 9, std=0.06)
    wqkv = synth.weights_f32(bits)["enc.0.attn.wqkv"].copy()
    wqkv[:256] *= 3.0
    bits["enc.0.attn.wqkv"] = synth.f32_to_bf16_bits(wqkv)
    model = orc.Model(desc, synth.weights_f32(bits))
    src = synth.random_tokens(S, "src", (4, S), desc)
    ses = sd.Session(4, 4, S, 16, fill=0xFF)
    ses.bind_model(sd.SPECDEC_VERIFIER, desc, ses.upload_weights(bits))
    sd.specdec_begin(ses.ctx, 4, 8)
    sd.specdec_encode(ses.ctx, ses.i32(src), ses.i32(np.asarray(lens, np.int32)))
    mem = torch.zeros((4, S, desc.d_model), dtype=torch.bfloat16, device=ses.device)
    sd.specdec_get_memory(ses.ctx, sd.SPECDEC_VERIFIER, mem)
    torch.cuda.synchronize()
    got = mem.float().cpu().numpy()
    for b, n in enumerate(lens):
        want = orc.encode(model, [int(t) for t in src[b, :n]])
        # queries and keys are rounded to 2^-9: scores (standard deviation 4) to some 4 * 2^-8, the attention output by that share
        assert np.sqrt(np.mean((got[b, :n] - want) ** 2)) <= 1e-2, (b, n)
        assert np.abs(got[b, :n] - want).max() <= 1e-1, (b, n)
    ses.close()
