"""Prefill passes of few rows (d_model 512) as one kernel, each XCD on sequences of its own, which ends where the last layer's keys and values are
stored: what it caches against the oracle, for streams of different lengths, empty ones among them; waits given up; more rows than it takes."""
import time

import numpy as np
import pytest
import torch

import cases
import gpu_harness as gh
from paper_2203_16487_amd import binding as sd
from paper_2203_16487_amd import synth
from test_gpu_one_kernel import check, desc, resident_launches

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("passes,B,lo,hi,layers", [
    (1, 1, 1, 1, 2),         # one row
    (1, 1, 17, 17, 3),       # two row tiles, two query tiles
    (1, 6, 0, 3, 1),         # one layer: its keys and values alone; empty streams
    (1, 1, 80, 80, 2),       # five: the most of one sequence
    (0, 1, 81, 81, 2),       # launches
    (1, 9, 56, 56, 2),       # 112 rows of an XCD, seven: the most
    (1, 4, 112, 112, 2),
    (0, 4, 113, 113, 2),
    (1, 12, 0, 50, 2),
    (1, 40, 0, 20, 2),
])
def test_what_is_cached(passes, B, lo, hi, layers):
    case = cases.make_verify_case(desc(512, layers), seed=800 + B + hi, B=B, S=20, k=4, beta=3, tau=1.0, len_lo=lo, len_hi=hi, drafts="random",
                                  ragged_src=True)
    cases.run_oracle(case)
    ses = gh.open_verifier(case, fill=0xFF)
    outs = []
    for give_up in (0, 1, 0) if passes else (0,):
        sd.specdec_configure(ses.ctx, sd.SPECDEC_OPT_GIVE_UP_WAITS, give_up)
        sd.specdec_set_stream(ses.ctx, ses.i32(case.tokens), ses.i32(case.lens))
        n, _ = resident_launches(ses, lambda: sd.specdec_prefill(ses.ctx, sd.SPECDEC_VERIFIER))
        assert n == passes
        K, V = gh.gpu_cache(ses, case, max(case.L_max, 1))
        sd.specdec_configure(ses.ctx, sd.SPECDEC_OPT_GIVE_UP_WAITS, 0)
        out = gh.gpu_verify(ses, case)
        check(case, out)
        for b, st in enumerate(case.states):
            j = int(case.lens[b])
            for l in range(layers):
                assert np.abs(K[l, b, :j] - st.K[l][:j]).max(initial=0) <= 3e-2, (b, l)
                assert np.abs(V[l, b, :j] - st.V[l][:j]).max(initial=0) <= 3e-2, (b, l)
        live = np.arange(max(case.L_max, 1))[None, :] < case.lens[:, None]
        outs.append((K * live[None, :, :, None], V * live[None, :, :, None], out["logits"]))
    for o in outs[1:]:
        assert all(np.array_equal(a, b) for a, b in zip(o, outs[0]))
    ses.close()


def test_behind_a_cache():
    """A stream that grows behind cached rows (commits of plain steps rolled into one prefill after set_stream and a shorter cache)."""
    case = cases.make_verify_case(desc(512), seed=850, B=5, S=30, k=4, beta=3, tau=1.0, len_lo=20, len_hi=60, drafts="random", ragged_src=True)
    cases.run_oracle(case)
    ses = gh.open_verifier(case, fill=0xFF)
    n = case.lens - np.array([0, 1, 7, 19, 20])
    L = max(case.L_max, 1)
    K, V = cases.oracle_flat_cache(case, L)
    sd.specdec_set_stream(ses.ctx, ses.i32(case.tokens), ses.i32(case.lens))
    sd.specdec_load_cache(ses.ctx, sd.SPECDEC_VERIFIER, ses.bf16(K), ses.bf16(V), ses.i32(n))
    launches, _ = resident_launches(ses, lambda: sd.specdec_prefill(ses.ctx, sd.SPECDEC_VERIFIER))
    assert launches == 1
    check(case, gh.gpu_verify(ses, case))
    ses.close()


def test_bound_beyond_what_a_stream_can_have():
    """Four commits without a draft between them: the bound on what the drafter has not cached is 45 tokens, a stream has 34 at most.  The prefill that
    the draft begins with has places for these, and caches what one after set_stream does."""
    B, k, max_tgt, seed = 9, 10, 33, 860
    vd, dd = (synth.ModelDesc(0, layers, 512, 8, 2048, 1003, 20, 64).resolved() for layers in (1, 2))
    ses = sd.Session(16, k, 20, max_tgt, fill=0xFF)
    ses.bind_model(sd.SPECDEC_VERIFIER, vd, ses.upload_weights(synth.make_weights(vd, seed, std=0.02)))
    ses.bind_model(sd.SPECDEC_DRAFTER, dd, ses.upload_weights(synth.make_weights(dd, seed, tag="drafter", std=0.02)))
    dev = ses.device
    sd.specdec_begin(ses.ctx, B, 30)
    for role, tag in ((sd.SPECDEC_VERIFIER, 1), (sd.SPECDEC_DRAFTER, 2)):
        sd.specdec_set_memory(ses.ctx, role, ses.bf16(synth.make_memory(seed + tag, B, 20, 512)), ses.i32(np.full(B, 20)))
    acc, nxt, out_len = (torch.zeros(B, dtype=torch.int32, device=dev) for _ in range(3))
    for i in range(4):
        sd.specdec_verify(ses.ctx, ses.i32(synth.random_tokens(seed + i, "drafts", (B, k), vd, full_vocab=True)), k, 3, 1.0, acc, nxt)
        sd.specdec_commit(ses.ctx, acc, nxt)
    toks = torch.zeros((B, max_tgt), dtype=torch.int32, device=dev)
    sd.specdec_get_output(ses.ctx, toks, out_len)
    dr = torch.zeros((B, k), dtype=torch.int32, device=dev)
    z = torch.zeros((B, k, dd.vocab), dtype=torch.float32, device=dev)
    L = int(out_len.max()) + 1
    K, V = (torch.zeros((2, B, L, 512), dtype=torch.bfloat16, device=dev) for _ in range(2))
    got = []
    for again in (False, True):
        if again:
            stream = torch.cat([torch.full((B, 1), dd.bos_id, dtype=torch.int32, device=dev), toks[:, :L - 1]], 1).contiguous()
            sd.specdec_set_stream(ses.ctx, stream, out_len)
            sd.specdec_configure(ses.ctx, sd.SPECDEC_OPT_SMALL_BATCH_KERNELS, 0)
            sd.specdec_prefill(ses.ctx, sd.SPECDEC_DRAFTER)
        n, _ = resident_launches(ses, lambda: sd.specdec_draft(ses.ctx, k, dr, z))
        assert n == (0 if again else 1)
        sd.specdec_get_cache(ses.ctx, sd.SPECDEC_DRAFTER, K, V)
        live = (torch.arange(L, device=dev)[None, :] <= out_len[:, None])[None, :, :, None]
        got.append([(t.float() * live).cpu().numpy() for t in (K, V)] + [z.cpu().numpy()])
    ses.close()
    for a, b in zip(*got):
        assert np.isfinite(a).all() and np.abs(a - b).max() <= 3e-2


@pytest.mark.parametrize("lens,T", [
    ([0, 12, 5], 12),                     # an XCD's only stream is empty; eight units of attention
    ([0] * 8, 16),
    ([0, 0, 7, 16, 0, 3, 1, 0, 9], 16),   # two empty ones to an XCD, and one
    ([0], 80),                            # places of five query tiles
])
def test_streams_without_rows(lens, T):
    """No row of the pass to an XCD, in a model of six layers, whose exchange buffers are used in turn: waits end (one in vain takes 0.1 s), and what is
    cached and verified for the others is what launches give."""
    B, lens = len(lens), np.array(lens, np.int32)
    case = cases.make_verify_case(desc(512, 6), seed=870 + B, B=B, S=20, k=4, beta=3, tau=1.0, len_lo=T, len_hi=T, ragged_src=True)
    ses = gh.open_verifier(case, fill=0xFF)
    outs = []
    for small in (0, 1):
        sd.specdec_configure(ses.ctx, sd.SPECDEC_OPT_SMALL_BATCH_KERNELS, small)
        for n in [case.lens] + [lens] * 20:   # (first with rows everywhere: kernels loaded)
            sd.specdec_set_stream(ses.ctx, ses.i32(case.tokens), ses.i32(n))
            torch.cuda.synchronize()
            t = time.perf_counter()
            launches, _ = resident_launches(ses, lambda: sd.specdec_prefill(ses.ctx, sd.SPECDEC_VERIFIER))
            torch.cuda.synchronize()
            assert launches == small
            if n is lens:
                assert time.perf_counter() - t < 0.05
        K, V = gh.gpu_cache(ses, case, T)
        live = (np.arange(T)[None, :] < lens[:, None])[None, :, :, None]
        outs.append((K * live, V * live, gh.gpu_verify(ses, case)["logits"]))
    ses.close()
    for a, b, tol in zip(*outs, (3e-2, 3e-2, 2 * max(2e-2, 0.04 * float(outs[0][2].std())))):   # (logits: either within half of it of the oracle's)
        assert np.isfinite(a).all() and np.abs(a - b).max() <= tol
