"""A drafter's pass of few rows (d_model 512, at least 200 drafts) as one kernel, each XCD on sequences of its own: row tiles and their remainders, stream rows of
different numbers a sequence, slots beyond one tile of 16 queries and beyond a chunk of keys, against the oracle, and the launches of passes of fewer
drafts; caches loaded short of the stream, waits given up, replays of a captured pass, and the launches it takes with the kernels for small batches off."""
import numpy as np
import pytest
import torch

import specdec_oracle as orc
import test_gpu_draft_loop as dl
import test_gpu_parity_extra as px
from paper_2203_16487_amd import binding as sd
from paper_2203_16487_amd import synth
from test_gpu_one_kernel import FP8_KV, resident_launches

pytestmark = pytest.mark.gpu
STD = 0.02


def model(seed=31):
    dd = synth.ModelDesc(1, 2, 512, 8, 2048, 1003, 300, 330).resolved()
    db = synth.make_weights(dd, seed, tag="drafter", std=STD)
    return dd, db, orc.Model(dd, synth.weights_f32(db))


@pytest.mark.parametrize("one,B,k,S,j,prefill", [
    # j: stream lengths; without a prefill all j + 1 rows are the pass's own.
    # launches: fewer than 200 drafts
    (0, 1, 1, 5, (0, 0), False),        # one stream row, one slot
    (0, 1, 15, 40, (31, 31), True),
    (0, 1, 16, 40, (15, 15), False),    # 16 + 16: the slots are the second query tile
    (0, 3, 20, 90, (0, 12), False),
    (0, 1, 31, 33, (31, 31), False),    # 32 + 31: the most a sequence can have
    (0, 9, 10, 40, (0, 75), True),
    (0, 2, 12, 260, (250, 290), True),
    # one kernel: rows of an XCD, row tiles
    (1, 7, 31, 5, (0, 0), False),       # 1 + 31, two; one sequence to an XCD
    (1, 40, 5, 20, (31, 31), True),     # 30, two
    (1, 16, 15, 40, (0, 31), True),     # 32, two: a sequence's places are a query tile
    (1, 25, 8, 40, (0, 75), True),      # 36 and 27, three and two
    (1, 7, 29, 90, (0, 12), False),     # up to 42, three; one sequence to an XCD
    (1, 8, 25, 20, (0, 25), False),     # up to 51, four; places of two query tiles without rows
    (1, 24, 10, 30, (0, 10), False),    # up to 63, four
    (1, 40, 10, 64, (20, 140), True),   # 55, four
    (1, 64, 7, 70, (0, 60), True),      # 64, four
    (1, 8, 31, 33, (31, 31), False),    # 32 + 31, four: the most a sequence can have
    (1, 16, 16, 40, (15, 15), False),   # 2 x (16 + 16), four: the slots are the second query tile
    (1, 11, 20, 90, (0, 12), False),    # up to 66, five
    (1, 17, 12, 260, (250, 290), True), # several chunks of keys a wave
])
def test_against_oracle(one, B, k, S, j, prefill):
    dd, db, dm = model()
    lens = synth.random_lengths(100 + B + k, "len", B, *j)
    lens[0] = j[1]
    px.drafter_pass_case(dd, db, dm, B=B, S_max=S, k=k, lens=lens, seed=100 + B, prefill=prefill, max_tgt=330,
                         sample=sorted({0, B // 2, B - 1}) if B > 3 else None, one=one)


def open_pass(B, k, j, seed, options=None, S=30, ver=None):
    dd, db, dm = model()
    lens = synth.random_lengths(seed, "len", B, *j)
    toks = synth.random_tokens(seed, "stream", (B, int(lens.max()) + 1), dd)
    toks[:, 0] = dd.bos_id
    ses = dl.open_session(B, k, S, 330, ver=ver, dr=(dd, db), options=options)
    sd.specdec_begin(ses.ctx, B, 100)
    sd.specdec_encode(ses.ctx, ses.i32(synth.random_tokens(seed, "src", (B, S), dd)), ses.i32(synth.random_lengths(seed, "src_len", B, 2, S)))
    sd.specdec_set_stream(ses.ctx, ses.i32(toks), ses.i32(lens))
    return ses, dd, toks, lens


def draft(ses, dd, B, k, lens, fresh):
    """Drafts and slot logits of a pass; `fresh`: its rows are all of the stream's (else those of a pass behind another one)."""
    if fresh:
        sd.specdec_rewind(ses.ctx, ses.i32(lens))
    dr = torch.full((B, k), -1, dtype=torch.int32, device=ses.device)
    z = torch.full((B, k, dd.vocab), float("nan"), dtype=torch.float32, device=ses.device)
    sd.specdec_draft(ses.ctx, k, dr, z)
    torch.cuda.synchronize()
    return dr.cpu().numpy(), z.cpu().numpy()


@pytest.mark.parametrize("B,k,j,options", [(8, 25, (3, 3), {}), (20, 10, (0, 10), {}), (24, 10, (0, 10), {}), (23, 9, (0, 9), FP8_KV)])
def test_one_launch_and_waits_given_up(B, k, j, options):
    """One launch of the decoder; the same bits from its second run; with the option off separate launches, the same but for the order of sums."""
    ses, dd, toks, lens = open_pass(B, k, j, 200 + B, options)
    n, want = resident_launches(ses, lambda: draft(ses, dd, B, k, lens, False))
    assert n == 1
    again = draft(ses, dd, B, k, lens, True)     # (nothing left to ingest but what the rewind cut)
    for give_up in (1, 0):
        sd.specdec_configure(ses.ctx, sd.SPECDEC_OPT_GIVE_UP_WAITS, give_up)
        got = draft(ses, dd, B, k, lens, True)
        assert np.array_equal(got[1], again[1]), give_up
        assert np.array_equal(got[0], again[0]), give_up
    sd.specdec_configure(ses.ctx, sd.SPECDEC_OPT_SMALL_BATCH_KERNELS, 0)
    n, other = resident_launches(ses, lambda: draft(ses, dd, B, k, lens, True))
    ses.close()
    assert n == 0
    for z in (want[1], again[1]):
        assert np.abs(z - other[1]).max() <= px.LOGIT_TOL


@pytest.mark.parametrize("B,k,one", [(1, 5, 0), (19, 10, 0), (22, 9, 0), (20, 10, 1)])
def test_fewer_than_200_drafts_keep_the_launches(B, k, one):
    ses, dd, _, lens = open_pass(B, k, (0, 9), 300 + B)
    n, _ = resident_launches(ses, lambda: draft(ses, dd, B, k, lens, False))
    ses.close()
    assert n == one


def test_short_cache_gives_pad_drafts():
    """A cache loaded more than a row short of the stream: no place for that sequence's slots; the others' are what they were."""
    B, k = 20, 10
    ses, dd, toks, lens = open_pass(B, k, (6, 9), 77)
    sd.specdec_prefill(ses.ctx, sd.SPECDEC_DRAFTER)
    L = int(lens.max()) + 1
    K = torch.zeros((dd.dec_layers, B, L, dd.d_model), dtype=torch.bfloat16, device=ses.device)
    V = torch.zeros_like(K)
    sd.specdec_get_cache(ses.ctx, sd.SPECDEC_DRAFTER, K, V)
    full = draft(ses, dd, B, k, lens, False)[0]
    for cut in ([2], [0, 1, 2, 3]):
        n = lens.copy()
        n[cut] -= 2
        sd.specdec_set_stream(ses.ctx, ses.i32(toks), ses.i32(lens))
        sd.specdec_load_cache(ses.ctx, sd.SPECDEC_DRAFTER, K, V, ses.i32(n))
        launches, (got, _) = resident_launches(ses, lambda: draft(ses, dd, B, k, lens, False))
        assert launches == 1
        assert (got[cut] == dd.pad_id).all()
        rest = [b for b in range(B) if b not in cut]
        assert np.array_equal(got[rest], full[rest])
    ses.close()


def test_replays_of_a_captured_pass():
    """set_prefix, draft and its statistics as a graph: every replay, other work between them, has the eager pass's bits.  (One kernel in a context
    that has captured verification.)"""
    B, k = 20, 10
    vd = synth.ModelDesc(1, 1, 512, 8, 2048, 1003, 300, 330).resolved()
    ses, dd, toks, lens = open_pass(B, k, (12, 40), 78, ver=(vd, synth.make_weights(vd, 32, std=STD)))
    sd.specdec_prefill(ses.ctx, sd.SPECDEC_VERIFIER)
    acc, nxt = ses.i32(np.zeros(B)), ses.i32(np.zeros(B))
    sd.specdec_prefill(ses.ctx, sd.SPECDEC_DRAFTER)
    L = int(lens.max())
    K = torch.zeros((dd.dec_layers, B, L, dd.d_model), dtype=torch.bfloat16, device=ses.device)
    V = torch.zeros_like(K)
    sd.specdec_get_cache(ses.ctx, sd.SPECDEC_DRAFTER, K, V)
    t, n = ses.i32(toks), ses.i32(lens)
    dr = torch.zeros((B, k), dtype=torch.int32, device=ses.device)
    z = torch.zeros((B, k, dd.vocab), dtype=torch.float32, device=ses.device)

    def call():
        sd.specdec_set_prefix(ses.ctx, sd.SPECDEC_DRAFTER, t, n, K, V)
        sd.specdec_draft(ses.ctx, k, dr, z)

    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        verifies = torch.cuda.CUDAGraph()
        sd.specdec_verify(ses.ctx, None, 0, 1, 0.0, acc, nxt)
        side.synchronize()
        with torch.cuda.graph(verifies, stream=side):
            sd.specdec_verify(ses.ctx, None, 0, 1, 0.0, acc, nxt)
        launches, _ = resident_launches(ses, call)
        assert launches == 1
        side.synchronize()
        want = dr.clone(), z.clone()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            call()
        for _ in range(4):
            dr.zero_(); z.zero_()
            graph.replay()
            side.synchronize()
            assert torch.equal(dr, want[0]) and torch.equal(z, want[1])
            assert torch.isfinite(torch.randn(1000, device=ses.device).cumsum(0)).all()
    ses.close()
