"""How many stream tokens the drafter's pass has places for: sequences that a short cache has left behind catch up also where little is committed, and a
captured pass serves what is committed between its replays, whatever the blocks before its capture."""
import numpy as np
import torch
import pytest

from paper_2203_16487_amd import binding as sd
from test_gpu_draft_loop import make_models, open_session
from paper_2203_16487_amd import synth

pytestmark = pytest.mark.gpu
B, K_MAX, S = 3, 10, 8


def opened(seed, j):
    ver, dr = make_models(seed)
    ses = open_session(B, K_MAX, S, 64, ver=ver[:2], dr=dr[:2])
    sd.specdec_begin(ses.ctx, B, 60)
    sd.specdec_encode(ses.ctx, ses.i32(synth.random_tokens(seed, "src", (B, S), dr[0])), ses.i32(np.full(B, S)))
    toks = synth.random_tokens(seed, "stream", (B, j + 1), dr[0])
    toks[:, 0] = dr[0].bos_id
    sd.specdec_set_stream(ses.ctx, ses.i32(toks), ses.i32(np.full(B, j)))
    sd.specdec_prefill(ses.ctx, sd.SPECDEC_VERIFIER)
    out = {"dr": torch.zeros((B, K_MAX), dtype=torch.int32, device=ses.device),
           "z": torch.zeros((B, K_MAX, dr[0].vocab), dtype=torch.float32, device=ses.device),
           "acc": ses.i32(np.zeros(B)), "nxt": ses.i32(np.zeros(B))}
    return ses, dr[0], toks, out


def step(ses, desc, out, k, a, tokens):
    """One verification pass of k drafts of which a are committed, and the token behind them; tokens: [B, k + 1]."""
    sd.specdec_verify(ses.ctx, ses.i32(tokens[:, :k]) if k else None, k, 1, 0.0, out["acc"], out["nxt"])
    sd.specdec_commit(ses.ctx, ses.i32(np.full(B, a)), ses.i32(tokens[:, k]))


def expected(seed, stream):
    """Slot logits of a fresh context's pass behind these streams."""
    ses, desc, _, out = opened(seed, 1)
    sd.specdec_set_stream(ses.ctx, ses.i32(stream), ses.i32(np.full(B, stream.shape[1] - 1)))
    sd.specdec_draft(ses.ctx, K_MAX, out["dr"], out["z"])
    z = out["z"].cpu().numpy()
    ses.close()
    return z


def same(out, z):
    # (equal but for the order of sums: bf16 operands, logits of magnitude 1)
    assert np.abs(out["z"].cpu().numpy() - z).max() <= 2e-2
    assert np.array_equal(out["dr"].cpu().numpy(), out["z"].cpu().numpy().argmax(-1))


@pytest.mark.parametrize("short", [1, 4])
def test_a_short_cache_is_made_up_for(short):
    """A cache loaded short of the stream gives pad drafts; behind plain steps, which append one token each, the next pass has the drafts again."""
    seed, j = 21, 9
    ses, desc, toks, out = opened(seed, j)
    sd.specdec_prefill(ses.ctx, sd.SPECDEC_DRAFTER)
    K = torch.zeros((desc.dec_layers, B, j, desc.d_model), dtype=torch.bfloat16, device=ses.device)
    V = torch.zeros_like(K)
    sd.specdec_get_cache(ses.ctx, sd.SPECDEC_DRAFTER, K, V)
    sd.specdec_set_stream(ses.ctx, ses.i32(toks), ses.i32(np.full(B, j)))
    sd.specdec_prefill(ses.ctx, sd.SPECDEC_VERIFIER)
    sd.specdec_load_cache(ses.ctx, sd.SPECDEC_DRAFTER, K, V, ses.i32(np.full(B, j - short)))
    sd.specdec_draft(ses.ctx, K_MAX, out["dr"], out["z"])
    assert (out["dr"] == desc.pad_id).all()
    more = synth.random_tokens(seed, "more", (B, 2), desc)
    for i in range(2):
        step(ses, desc, out, 0, 0, more[:, i:i + 1])
        sd.specdec_draft(ses.ctx, K_MAX, out["dr"], out["z"])
        same(out, expected(seed, np.concatenate([toks, more[:, :i + 1]], 1)))
    ses.close()


def test_a_captured_pass_behind_larger_blocks():
    """A drafter's pass captured behind a block of two, replayed behind a block of ten all of which is committed."""
    seed, j = 22, 5
    ses, desc, toks, out = opened(seed, j)
    blocks = synth.random_tokens(seed, "blocks", (B, 3 + 11 + 11), desc)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        sd.specdec_draft(ses.ctx, K_MAX, out["dr"], out["z"])
        step(ses, desc, out, 2, 2, blocks[:, :3])
        side.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            sd.specdec_draft(ses.ctx, K_MAX, out["dr"], out["z"])
        graph.replay()
        side.synchronize()
        same(out, expected(seed, np.concatenate([toks, blocks[:, :3]], 1)))
        for n in (14, 25):
            step(ses, desc, out, 10, 10, blocks[:, n - 11:n])
            graph.replay()
            side.synchronize()
            same(out, expected(seed, np.concatenate([toks, blocks[:, :n]], 1)))
    ses.close()
