"""The two models' encoders beside each other (specdec_encode with both bound): the bits of one after the other (which timed launches and a
stream without all compute units take), sources replaced behind the call, replays of a captured call, a context destroyed with one in flight."""
import numpy as np
import pytest
import torch

from paper_2203_16487_amd import binding as sd
from paper_2203_16487_amd import synth
from test_gpu_one_kernel import masked_stream

pytestmark = pytest.mark.gpu


def open_both(B, S, seed):
    vd = synth.ModelDesc(3, 1, 512, 8, 2048, 1000, S, 40).resolved()
    dd = synth.ModelDesc(5, 1, 256, 4, 1024, 1000, S, 40).resolved()
    ses = sd.Session(B, 4, S, 40)
    for role, d, tag in ((sd.SPECDEC_VERIFIER, vd, "verifier"), (sd.SPECDEC_DRAFTER, dd, "drafter")):
        ses.bind_model(role, d, ses.upload_weights(synth.make_weights(d, seed, tag=tag)))
    src = [ses.i32(synth.random_tokens(seed + i, "src", (B, S), vd)) for i in range(2)]
    lens = ses.i32(synth.random_lengths(seed, "src_len", B, 1, S))
    out = [torch.zeros((B, S, d.d_model), dtype=torch.bfloat16, device=ses.device) for d in (vd, dd)]
    z = torch.zeros((B, 1, vd.vocab), dtype=torch.float32, device=ses.device)
    dr = torch.zeros((B, 4), dtype=torch.int32, device=ses.device)
    zd = torch.zeros((B, 4, vd.vocab), dtype=torch.float32, device=ses.device)
    acc, nxt = ses.i32(np.zeros(B)), ses.i32(np.zeros(B))

    def call(s):
        sd.specdec_begin(ses.ctx, B, 10)
        sd.specdec_encode(ses.ctx, s, lens)
        for role, o in zip((sd.SPECDEC_VERIFIER, sd.SPECDEC_DRAFTER), out):
            sd.specdec_get_memory(ses.ctx, role, o)
        sd.specdec_verify(ses.ctx, None, 0, 1, 0.0, acc, nxt, z)
        sd.specdec_draft(ses.ctx, 4, dr, zd)

    def results():
        torch.cuda.synchronize()
        return [t.clone() for t in (*out, z, zd)]

    return ses, src, call, results


def same(a, b):
    return all(torch.equal(x, y) for x, y in zip(a, b))


@pytest.mark.parametrize("B,S", [(1, 1), (5, 37), (40, 128)])
def test_bits_of_one_after_the_other(B, S):
    ses, src, call, results = open_both(B, S, 11)
    sd.specdec_profile_select(ses.ctx, sd.KIND["gemm_qkv"])   # (timed: one after the other)
    want = []
    for s in src:
        call(s)
        want.append(results())
    sd.specdec_profile_select(ses.ctx, sd.KIND["none"])
    for i in (0, 1, 0):
        call(src[i])
        assert same(results(), want[i]), i
    tokens = src[0].clone()
    for i in (1, 0):            # the caller's next work may replace what the call reads
        tokens.copy_(src[i])
        call(tokens)
        tokens.fill_(7)
        assert same(results(), want[i]), i
    ses.close()


def test_replays_of_a_captured_call():
    ses, src, call, results = open_both(9, 50, 12)
    call(src[0])
    want = [results()]
    call(src[1])
    want.append(results())
    tokens = src[0].clone()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        call(tokens)
    for i in (0, 1, 1, 0):
        tokens.copy_(src[i])
        torch.cuda.synchronize()
        graph.replay()
        assert same(results(), want[i]), i
        torch.randn(1000, device=ses.device).sum().item()
    ses.close()


def test_stream_with_few_compute_units():
    """Such a stream takes them one after the other, on what it has."""
    ses, src, call, results = open_both(6, 40, 13)
    sd.specdec_configure(ses.ctx, sd.SPECDEC_OPT_SMALL_BATCH_KERNELS, 0)   # (the same decoder kernels on either stream)
    call(src[0])
    want = results()
    stream = masked_stream([0xffffffff] * 2 + [0] * 6)
    with torch.cuda.stream(stream):
        call(src[0])
        stream.synchronize()
        assert same(results(), want)
    ses.close()


def test_destroyed_with_a_call_in_flight():
    ses, src, call, results = open_both(40, 128, 14)
    call(src[0])
    want = results()
    call(src[1])
    call(src[0])
    sd.specdec_destroy(ses.ctx)   # (its buffers outlive it)
    ses.ctx = None
    assert same(results(), want)
