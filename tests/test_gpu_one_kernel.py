"""The decoder layers of a pass of few rows as one kernel (d_model 512 / 1024), over the whole GPU or per XCD: row tiles and their
remainders, queries beyond one tile of 16, key chunks split over the waves and not, a unit of attention per workgroup and per wave,
E4M3 weights and cross keys / values, against the oracle; waits given up; the path a second context takes; replays of a captured pass."""
import contextlib
import ctypes as C

import numpy as np
import pytest
import torch

import cases
import gpu_harness as gh
from paper_2203_16487_amd import binding as sd
from paper_2203_16487_amd import synth
import specdec_oracle as orc

pytestmark = pytest.mark.gpu


def desc(d, layers=2):
    return synth.ModelDesc(0, layers, d, d // 64, 4 * d, 1003, 64, 300).resolved()


def check(case, out):
    err = float(np.abs(out["logits"] - case.logits).max())
    exact, excused, bad = cases.compare_decisions(case, out["accept"], out["next"])
    assert err <= max(2e-2, 0.04 * float(case.logits.std())), err
    assert not bad, bad


FP8_W, FP8_KV = {sd.SPECDEC_OPT_FP8_WEIGHTS: 1}, {sd.SPECDEC_OPT_FP8_CROSS_KV: 1}


def masked_stream(words):
    """A stream whose kernels may use the compute units of this mask only."""
    path = next(line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64.so" in line)
    hip, handle = C.CDLL(path), C.c_void_p()
    assert hip.hipExtStreamCreateWithCUMask(C.byref(handle), C.c_uint32(len(words)), (C.c_uint32 * len(words))(*words)) == 0
    return torch.cuda.ExternalStream(handle.value)


@contextlib.contextmanager
def compute_units(n):
    """What is inside runs on a stream that may use n compute units (a multiple of 32; None: the default stream)."""
    if n is None:
        yield
        return
    torch.cuda.synchronize()
    stream = masked_stream([0xffffffff] * (n // 32) + [0] * (8 - n // 32))
    with torch.cuda.stream(stream):
        yield
    stream.synchronize()


@pytest.mark.parametrize("way,d,B,k,S,lo,hi,opts", [
    # per XCD, weights in place; rows of an XCD, row tiles
    ("xcd in place", 512, 1, 1, 5, 0, 0, {}),       # two rows, nothing cached
    ("xcd in place", 512, 1, 16, 40, 31, 31, {}),   # 17, two: a second query tile of one row
    ("xcd in place", 512, 2, 15, 200, 180, 220, {}),   # every wave has key chunks
    ("xcd in place", 512, 3, 15, 90, 20, 60, {}),   # 16, one
    ("xcd in place", 512, 9, 6, 40, 0, 75, {}),     # 14 and 7; 63 rows, the most
    ("xcd in place", 512, 63, 0, 20, 0, 40, {}),    # 8 and 7: plain steps
    ("xcd in place", 512, 3, 9, 50, 0, 40, FP8_KV),
    ("xcd in place", 512, 21, 2, 50, 0, 40, FP8_KV),   # 9 and 6; 63 rows
    # over the whole GPU
    ("gpu", 512, 3, 9, 50, 0, 40, FP8_W),
    ("gpu", 1024, 1, 25, 90, 57, 57, {}),
    ("gpu", 1024, 16, 3, 30, 0, 40, {}),            # 64 rows, the most on tiles of 16 rows
    ("gpu", 1024, 13, 4, 30, 0, 140, {}),           # 65 rows: tiles of 32, the last of one row
    ("gpu", 1024, 9, 10, 300, 0, 140, {}),          # 99 rows
    ("gpu", 1024, 64, 1, 40, 50, 70, {}),           # 128 rows, the most; two waves per unit
    ("gpu", 1024, 11, 10, 150, 100, 130, FP8_KV),
    ("gpu", 1024, 24, 4, 200, 60, 140, {}),         # four waves per unit, several chunks of keys each
    ("gpu", 1024, 1, 30, 33, 9, 9, {**FP8_W, **FP8_KV}),
    # per XCD; rows of an XCD, row tiles
    ("xcd", 512, 7, 10, 40, 0, 75, {}),             # 11 (one XCD has none), one
    ("xcd", 512, 64, 0, 40, 0, 75, {}),             # 8: plain steps
    ("xcd", 512, 7, 10, 40, 0, 75, FP8_KV),         # 11, one
    ("xcd", 512, 42, 2, 20, 0, 30, {}),             # 18 and 15, two
    ("xcd", 512, 43, 2, 20, 0, 30, {}),             # 18 and 15, more sequences with the larger share
    ("xcd", 512, 8, 16, 20, 0, 30, {}),             # 17, two; two query tiles a sequence
    ("xcd", 512, 32, 7, 20, 60, 90, {}),            # 32, two; a wave per unit of attention
    ("xcd", 512, 128, 1, 60, 0, 60, {}),            # 32: two rows a sequence, two rounds of units
    ("xcd", 512, 9, 12, 70, 0, 90, FP8_KV),         # 26 and 13, two
    ("xcd", 512, 9, 10, 50, 0, 40, FP8_W),          # 22 and 11: bf16 matrices, as in every pass of more than 32 rows
    ("xcd", 512, 32, 10, 64, 0, 64, {}),            # 44, three
    ("xcd", 512, 17, 14, 64, 0, 64, FP8_KV),        # 45 and 30, three
    ("xcd", 512, 37, 11, 70, 0, 130, {}),           # 60 and 48, four
    ("xcd", 512, 27, 15, 70, 0, 130, FP8_KV),       # 64 and 48, four
    ("xcd", 1024, 16, 10, 80, 0, 100, {}),          # 22, two
    ("xcd", 1024, 17, 8, 80, 0, 140, {}),           # 27 and 18, two
    ("xcd", 1024, 17, 8, 80, 0, 140, FP8_KV),
    ("xcd", 1024, 19, 10, 120, 11, 100, FP8_KV),    # 33 and 22, three
    ("xcd", 1024, 32, 10, 60, 0, 100, {}),          # 44, three
    ("xcd", 1024, 16, 31, 40, 0, 90, {}),           # 64, four: 512 rows, the most
    ("xcd", 1024, 17, 20, 45, 30, 90, FP8_KV),      # 63 and 42, four; two query tiles a sequence
])
def test_against_oracle(way, d, B, k, S, lo, hi, opts):
    case = cases.make_verify_case(desc(d), seed=d + 10 * B + k, B=B, S=S, k=k, beta=3, tau=1.0, len_lo=lo, len_hi=hi, drafts="random",
                                  ragged_src=True, fp8=sd.SPECDEC_OPT_FP8_WEIGHTS in opts and B * (k + 1) <= 32,
                                  fp8_kv=sd.SPECDEC_OPT_FP8_CROSS_KV in opts)
    cases.run_oracle(case)
    ses = gh.open_verifier(case, k_max=max(k, 1), options=opts, fill=0xFF)
    out = gh.gpu_verify(ses, case)
    again = gh.gpu_verify(ses, case)
    L = case.L_max + k + 1
    K, V = gh.gpu_cache(ses, case, L)
    assert sd.specdec_decoder_way(ses.ctx) == way
    ses.close()
    check(case, out)
    assert np.array_equal(out["logits"], again["logits"])
    for b, st in enumerate(case.states):
        j = int(case.lens[b])
        for l in range(case.desc.dec_layers):
            assert np.abs(K[l, b, j:j + k + 1] - st.K[l][j:j + k + 1]).max() <= 3e-2, (b, l)
            assert np.abs(V[l, b, j:j + k + 1] - st.V[l][j:j + k + 1]).max() <= 3e-2, (b, l)


@pytest.mark.parametrize("way,cus,B,k,S,lo,hi,opts", [
    ("gpu", 128, 1, 5, 32, 16, 16, {}),             # 104 workgroups
    ("gpu", 224, 1, 16, 40, 31, 31, {}),            # 17 rows: a second query tile of one row; 208 workgroups
    ("gpu", 224, 2, 15, 200, 180, 220, {}),         # every wave has key chunks
    ("gpu", 224, 3, 15, 90, 20, 60, {}),            # 48 rows, the most: three row tiles, items of four column tiles; 216
    ("gpu", 224, 2, 16, 60, 0, 75, FP8_KV),         # 34: the last row tile of two rows; 224
    ("gpu", 224, 4, 7, 50, 0, 40, FP8_KV),          # 32; 224
    ("gpu", 224, 16, 0, 50, 0, 40, {}),             # plain steps: 16 rows; 224
    ("launches", 224, 8, 4, 50, 0, 40, {}),         # 40: 256
    ("launches", 224, 7, 6, 50, 0, 40, {}),         # 49 rows
    ("launches", 192, 1, 16, 40, 31, 31, {}),
])
def test_against_oracle_on_fewer_compute_units(way, cus, B, k, S, lo, hi, opts):
    """bf16 weights of d_model 512 go over the whole GPU where the stream has fewer compute units than there are, but as many as the kernel has
    workgroups; given up, the kernel behind it gives the same bits."""
    case = cases.make_verify_case(desc(512), seed=512 + cus + 10 * B + k, B=B, S=S, k=k, beta=3, tau=1.0, len_lo=lo, len_hi=hi, drafts="random",
                                  ragged_src=True, fp8_kv=sd.SPECDEC_OPT_FP8_CROSS_KV in opts)
    cases.run_oracle(case)
    L = case.L_max + k + 1
    with compute_units(cus):
        ses = gh.open_verifier(case, k_max=max(k, 1), options=opts, fill=0xFF)
        sd.specdec_profile_select(ses.ctx, sd.KIND["resident"])
        out = gh.gpu_verify(ses, case)
        ms, n = sd.specdec_profile_read(ses.ctx)
        assert sd.specdec_decoder_way(ses.ctx) == way and n == (way == "gpu")
        assert ms < 50                                 # no wait ended at its bound
        K, V = gh.gpu_cache(ses, case, L)
        for give_up in (0, 1, 0):
            sd.specdec_configure(ses.ctx, sd.SPECDEC_OPT_GIVE_UP_WAITS, give_up)
            got = gh.gpu_verify(ses, case)
            for key in ("logits", "accept", "next", "stats"):
                assert np.array_equal(got[key], out[key]), (give_up, key)
            for x, y in zip(gh.gpu_cache(ses, case, L), (K, V)):
                for b, j in enumerate(case.lens):
                    assert np.array_equal(x[:, b, :j + k + 1], y[:, b, :j + k + 1])
        ses.close()
    check(case, out)
    for b, st in enumerate(case.states):
        j = int(case.lens[b])
        for l in range(case.desc.dec_layers):
            assert np.abs(K[l, b, j:j + k + 1] - st.K[l][j:j + k + 1]).max() <= 3e-2, (b, l)
            assert np.abs(V[l, b, j:j + k + 1] - st.V[l][j:j + k + 1]).max() <= 3e-2, (b, l)


@pytest.mark.parametrize("B,k", [(2, 5), (9, 10)])   # per XCD: weights in place; 99 rows
def test_two_contexts_and_replays(B, k):
    case = cases.make_verify_case(desc(512), seed=5, B=B, S=30, k=k, beta=3, tau=1.0, len_lo=3, len_hi=20, drafts="greedy",
                                  ragged_src=True)
    cases.run_oracle(case)
    first = gh.open_verifier(case, fill=0xFF)
    out = gh.gpu_verify(first, case)
    check(case, out)
    second = gh.open_verifier(case, fill=0xFF)
    assert np.array_equal(gh.gpu_verify(second, case)["logits"], out["logits"])
    other = torch.cuda.Stream()
    other.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(other):                    # (two streams: other kernels than the first context's)
        check(case, gh.gpu_verify(second, case))
    other.synchronize()
    second.close()
    d, acc, nxt = first.i32(case.drafts), torch.zeros(B, dtype=torch.int32, device="cuda"), torch.zeros(B, dtype=torch.int32, device="cuda")
    logits = torch.zeros((B, k + 1, case.desc.vocab), dtype=torch.float32, device="cuda")
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        sd.specdec_verify(first.ctx, d, case.k, case.beta, case.tau, acc, nxt, logits)
    for _ in range(4):
        logits.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(logits.cpu().numpy(), out["logits"])
        assert acc.cpu().tolist() == out["accept"].tolist() and nxt.cpu().tolist() == out["next"].tolist()
        assert np.array_equal(gh.gpu_verify(first, case)["logits"], out["logits"])
    first.close()


@pytest.mark.parametrize("way,d,B,k,S,lo,hi,opts", [
    # per XCD, weights in place
    ("xcd in place", 512, 1, 5, 32, 16, 16, {}),
    ("xcd in place", 512, 2, 15, 200, 180, 220, {}),   # every wave with key chunks
    ("xcd in place", 512, 9, 6, 40, 0, 75, {}),     # 63 rows, 14 and 7 of an XCD
    ("xcd in place", 512, 63, 0, 20, 0, 40, {}),
    # over the whole GPU
    ("gpu", 512, 1, 5, 32, 16, 16, FP8_W),
    ("gpu", 512, 2, 15, 200, 150, 180, FP8_W),      # a unit of attention per workgroup, every wave with key chunks
    ("gpu", 1024, 64, 1, 40, 50, 70, {}),           # more units than workgroups, items of 32 rows
    ("gpu", 1024, 11, 10, 150, 100, 130, FP8_KV),
    ("gpu", 1024, 1, 30, 33, 9, 9, {**FP8_W, **FP8_KV}),
    # per XCD; rows of an XCD
    ("xcd", 512, 9, 10, 40, 0, 75, {}),             # 22 and 11: one row tile in use, and two
    ("xcd", 512, 42, 2, 20, 0, 30, {}),             # 18 and 15
    ("xcd", 512, 32, 7, 20, 60, 90, {}),            # 32
    ("xcd", 512, 32, 10, 64, 0, 64, FP8_KV),        # 44
    ("xcd", 512, 37, 11, 70, 0, 130, {}),           # 60 and 48: all four row tiles, residual of the fourth
    ("xcd", 1024, 17, 8, 80, 0, 140, {}),           # 27 and 18
    ("xcd", 1024, 32, 10, 60, 0, 100, {}),          # 44
    ("xcd", 1024, 17, 20, 45, 30, 90, FP8_KV),      # 63 and 42; two query tiles a sequence
])
def test_waits_given_up(way, d, B, k, S, lo, hi, opts):
    """Waits of the kernel given up at once (per XCD: at their bound, as a workgroup of every group is missing, or with weights in place at
    their first look at the flag; either way it ends with half of its results missing): the kernel behind it computes the pass, to the
    last bit as the waiting one; so it does the next 63, which find the flag raised; then one waits again."""
    case = cases.make_verify_case(desc(d), seed=d + B, B=B, S=S, k=k, beta=3, tau=1.0, len_lo=lo, len_hi=hi, drafts="random",
                                  ragged_src=True, fp8=sd.SPECDEC_OPT_FP8_WEIGHTS in opts, fp8_kv=sd.SPECDEC_OPT_FP8_CROSS_KV in opts)
    cases.run_oracle(case)
    ses = gh.open_verifier(case, k_max=max(k, 1), options=opts, fill=0xFF)
    L = case.L_max + k + 1
    want, cache = gh.gpu_verify(ses, case), gh.gpu_cache(ses, case, L)
    assert sd.specdec_decoder_way(ses.ctx) == way
    check(case, want)
    sd.specdec_profile_select(ses.ctx, sd.KIND["resident"])
    times = []
    for give_up in (0, 1, 0):
        sd.specdec_configure(ses.ctx, sd.SPECDEC_OPT_GIVE_UP_WAITS, give_up)
        got = gh.gpu_verify(ses, case)
        times.append(sd.specdec_profile_read(ses.ctx)[0])
        if give_up:
            assert (times[-1] > 100) == (way == "xcd"), times   # (the 0.1 s that the header states)
        for key in ("logits", "accept", "next", "stats"):
            assert np.array_equal(got[key], want[key]), (give_up, key)
        for x, y in zip(gh.gpu_cache(ses, case, L), cache):
            for b, j in enumerate(case.lens):
                assert np.array_equal(x[:, b, :j + k + 1], y[:, b, :j + k + 1])
    for _ in range(65):
        got = gh.gpu_verify(ses, case, want_logits=False)
        assert np.array_equal(got["stats"], want["stats"])
    times.append(sd.specdec_profile_read(ses.ctx)[0] / 65)
    print(f"one-kernel decoder {times[0]:.3f} ms, given up {times[1]:.3f} ms, flag raised {times[2]:.3f} ms, mean of the next 65 {times[3]:.3f} ms")
    ses.close()


@pytest.mark.parametrize("d,B,k", [(512, 9, 10), (1024, 19, 10)])
def test_finished_sequences_per_xcd(d, B, k):
    """A pass after some sequences have ended, whole XCDs of them: theirs are computed and not reported, the others' as if alone; the same
    where waits are given up."""
    case = cases.make_verify_case(desc(d), seed=90 + d, B=B, S=30, k=k, beta=3, tau=1.0, len_lo=0, len_hi=20, drafts="random", ragged_src=True,
                                  cap_extra=1)
    cases.run_oracle(case)
    ses = gh.open_verifier(case, max_tgt=case.L_max + 2 * k + 8, fill=0xFF)
    check(case, gh.gpu_verify(ses, case))
    done = [b for b in range(B) if b < 2 or b % 3 == 0]
    nxt = [case.desc.eos_id if b in done else int(case.nxt[b]) for b in range(B)]
    sd.specdec_commit(ses.ctx, ses.i32(np.zeros(B)), ses.i32(nxt))
    outs = []
    for give_up in (0, 1):
        sd.specdec_configure(ses.ctx, sd.SPECDEC_OPT_GIVE_UP_WAITS, give_up)
        n, out = resident_launches(ses, lambda: gh.gpu_verify(ses, case))
        assert n == 1
        outs.append(out)
    ses.close()
    for key in ("logits", "accept", "next", "stats"):
        assert np.array_equal(outs[0][key], outs[1][key]), key
    for b, st in enumerate(case.states):
        if b in done:
            assert outs[0]["accept"][b] == 0 and outs[0]["next"][b] == case.desc.pad_id
            continue
        st.len += 1
        z = orc.verify_onepass(case.model, st, nxt[b], list(case.drafts[b]))
        assert float(np.abs(outs[0]["logits"][b] - z).max()) <= max(2e-2, 0.04 * float(z.std())), b


def test_each_decoder_gives_up_for_itself():
    """Passes of 9 rows read the weights in place, of 99 a copy of them, both per XCD: where one kind has given up its waits, the other still
    waits (its kernel takes some 40 us, 5 where it finds its flag raised)."""
    case = cases.make_verify_case(desc(512), seed=95, B=9, S=30, k=10, beta=3, tau=1.0, len_lo=0, len_hi=20, drafts="random", ragged_src=True)
    cases.run_oracle(case)
    ses = gh.open_verifier(case, fill=0xFF)
    acc, nxt, z = ses.i32(np.zeros(9)), ses.i32(np.zeros(9)), torch.zeros((9, 1, case.desc.vocab), dtype=torch.float32, device=ses.device)

    def few():
        sd.specdec_verify(ses.ctx, None, 0, 1, 0.0, acc, nxt, z)
        return z.cpu().numpy()

    def many():
        return gh.gpu_verify(ses, case)["logits"]

    want = {}
    for f, way in ((few, "xcd in place"), (many, "xcd")):
        want[f] = f()
        assert sd.specdec_decoder_way(ses.ctx) == way
    sd.specdec_profile_select(ses.ctx, sd.KIND["resident"])
    for given_up, other in ((few, many), (many, few)):
        sd.specdec_configure(ses.ctx, sd.SPECDEC_OPT_GIVE_UP_WAITS, 1)
        assert np.array_equal(given_up(), want[given_up])
        sd.specdec_configure(ses.ctx, sd.SPECDEC_OPT_GIVE_UP_WAITS, 0)
        sd.specdec_profile_read(ses.ctx)
        assert np.array_equal(other(), want[other])
        ms, n = sd.specdec_profile_read(ses.ctx)
        assert n == 1 and ms > 0.015, (given_up, ms)
        assert np.array_equal(given_up(), want[given_up])
        assert sd.specdec_profile_read(ses.ctx)[0] < 0.015
        restart(ses, case)                     # (a new run: no flag is raised)
    ses.close()


def resident_launches(ses, run):
    """How often the one-kernel decoder was launched by run(), and run()'s result."""
    sd.specdec_profile_select(ses.ctx, sd.KIND["resident"])
    out = run()
    n = sd.specdec_profile_read(ses.ctx)[1]
    sd.specdec_profile_select(ses.ctx, sd.KIND["none"])
    return n, out


def test_stream_with_few_compute_units():
    """The kernel's workgroups wait for each other: a stream that may not use as many compute units as there are workgroups
    takes separate launches."""
    case = cases.make_verify_case(desc(512), seed=42, B=42, S=20, k=2, beta=3, tau=1.0, len_lo=0, len_hi=30, drafts="random", ragged_src=True)
    cases.run_oracle(case)
    ses = gh.open_verifier(case, fill=0xFF)
    assert resident_launches(ses, lambda: gh.gpu_verify(ses, case))[0] == 1
    torch.cuda.synchronize()
    half = masked_stream([0xffffffff] * 4 + [0] * 4)
    with torch.cuda.stream(half):
        n, out = resident_launches(ses, lambda: gh.gpu_verify(ses, case))
    half.synchronize()
    assert n == 0
    check(case, out)
    ses.close()


def restart(ses, case):
    """A new run on the case's streams, memory and cache."""
    sd.specdec_begin(ses.ctx, case.B, 10 ** 6)
    sd.specdec_set_memory(ses.ctx, sd.SPECDEC_VERIFIER, ses.bf16(case.memory), ses.i32(case.src_len))
    sd.specdec_set_stream(ses.ctx, ses.i32(case.tokens), ses.i32(case.lens))
    K, V = cases.oracle_flat_cache(case, max(case.L_max, 1))
    sd.specdec_load_cache(ses.ctx, sd.SPECDEC_VERIFIER, ses.bf16(K), ses.bf16(V), ses.i32(case.lens))


@pytest.mark.parametrize("B,k", [(1, 5), (1, 11), (1, 12), (2, 5), (7, 10)])   # the fused small-batch kernels up to 12 rows, the general ones
def test_way_of_a_run_does_not_change(B, k):
    """A context refused the one-kernel decoder, because another one on another stream has it, keeps its separate launches when
    that one is gone, until its next run: a pass repeated gives the same bits."""
    case = cases.make_verify_case(desc(512), seed=50 + 10 * B + k, B=B, S=30, k=k, beta=3, tau=1.0, len_lo=3, len_hi=20,
                                  drafts="greedy", ragged_src=True)
    cases.run_oracle(case)
    first = gh.open_verifier(case, fill=0xFF)
    n, out = resident_launches(first, lambda: gh.gpu_verify(first, case))
    assert n == 1
    second = gh.open_verifier(case, fill=0xFF)
    other = torch.cuda.Stream()
    other.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(other):
        n, apart = resident_launches(second, lambda: gh.gpu_verify(second, case))
        assert n == 0
        check(case, apart)
        other.synchronize()
        first.close()
        n, again = resident_launches(second, lambda: gh.gpu_verify(second, case))
        assert n == 0 and np.array_equal(again["logits"], apart["logits"])
        restart(second, case)
        n, alone = resident_launches(second, lambda: gh.gpu_verify(second, case))
        assert n == 1 and np.array_equal(alone["logits"], out["logits"])
        other.synchronize()
        second.close()


def test_pass_in_flight_when_its_context_ends():
    """A context destroyed before its latest pass has run, and a pass of another context on another stream that may meet it:
    whichever way the two are completed, both are right."""
    case = cases.make_verify_case(desc(512), seed=60, B=7, S=30, k=10, beta=3, tau=1.0, len_lo=3, len_hi=20, drafts="greedy", ragged_src=True)
    cases.run_oracle(case)
    first, second = gh.open_verifier(case, fill=0xFF), gh.open_verifier(case, fill=0xFF)
    acc, nxt, d = first.i32(np.zeros(7)), first.i32(np.zeros(7)), first.i32(case.drafts)
    one, other = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    busy = torch.empty(1 << 28, dtype=torch.float32, device="cuda")
    with torch.cuda.stream(one):
        for _ in range(200):                           # some tens of milliseconds ahead of the pass
            busy.add_(1.0)
        sd.specdec_verify(first.ctx, d, case.k, case.beta, case.tau, acc, nxt)
    sd.specdec_destroy(first.ctx)                      # (what it points to stays)
    first.ctx = None
    with torch.cuda.stream(other):
        out = gh.gpu_verify(second, case)              # (waits for both)
    torch.cuda.synchronize()
    check(case, out)
    assert acc.cpu().tolist() == out["accept"].tolist()
    second.close()


@pytest.mark.parametrize("B,k", [(2, 5), (7, 10)])     # last sums left un-normalised (at most 32 rows) and not
def test_head_drafts_after_it(B, k):
    """The hidden states the kernel leaves to specdec_draft_heads, also where its waits were given up; SPECDEC_OPT_RESIDENT keeps
    refusing them after passes of at most 32 rows."""
    case = cases.make_verify_case(desc(512), seed=70 + B, B=B, S=30, k=k, beta=3, tau=1.0, len_lo=3, len_hi=20, drafts="greedy", ragged_src=True)
    cases.run_oracle(case)
    hb = synth.make_head_weights(case.desc, 3, 70, std=0.02)
    heads = [synth.weights_f32(h) for h in hb]
    ses = gh.open_verifier(case, fill=0xFF)
    stacked = ses.upload_weights({n: np.concatenate([h[n] for h in hb]) for n in ("w1", "b1", "w2", "b2")})   # (used in place)
    sd.specdec_bind_draft_heads(ses.ctx, 3, *stacked)
    z = torch.zeros((B, 3, case.desc.vocab), dtype=torch.float32, device=ses.device)
    drafts = ses.i32(np.zeros((B, 3)))
    for give_up in (0, 1):
        sd.specdec_configure(ses.ctx, sd.SPECDEC_OPT_GIVE_UP_WAITS, give_up)
        n, out = resident_launches(ses, lambda: gh.gpu_verify(ses, case))
        assert n == 1
        check(case, out)
        sd.specdec_draft_heads(ses.ctx, out["accept_t"], 3, drafts, z)
        torch.cuda.synchronize()
        for b in range(B):
            hidden = orc.verify_onepass(case.model, case.states[b], int(case.tokens[b, case.lens[b]]), list(case.drafts[b]), return_hidden=True)[1]
            want = orc.head_draft(case.model, heads, hidden[int(out["accept"][b])], return_logits=True)[1]
            assert float(np.abs(z[b].cpu().numpy() - want).max()) <= max(2e-2, 0.04 * float(want.std())), (give_up, b)
    sd.specdec_configure(ses.ctx, sd.SPECDEC_OPT_RESIDENT, 1)
    gh.gpu_verify(ses, case)
    if B * (k + 1) <= 32:
        with pytest.raises(sd.SpecDecError) as e:
            sd.specdec_draft_heads(ses.ctx, out["accept_t"], 3, drafts)
        assert e.value.code == sd.SPECDEC_ERR_BAD_STATE
    else:
        sd.specdec_draft_heads(ses.ctx, out["accept_t"], 3, drafts)
    ses.close()


@pytest.mark.parametrize("name", [1, 2])               # hipStreamLegacy, hipStreamPerThread
def test_default_streams_by_name(name):
    case = cases.make_verify_case(desc(512), seed=80, B=2, S=30, k=5, beta=3, tau=1.0, len_lo=3, len_hi=20, drafts="greedy", ragged_src=True)
    cases.run_oracle(case)
    ses = gh.open_verifier(case, fill=0xFF)
    out = gh.gpu_verify(ses, case)
    check(case, out)
    d, acc, nxt = ses.i32(case.drafts), ses.i32(np.zeros(2)), ses.i32(np.zeros(2))
    z = torch.zeros((2, 6, case.desc.vocab), dtype=torch.float32, device=ses.device)
    torch.cuda.synchronize()
    rc = sd.lib().specdec_verify(ses.ctx, d.data_ptr(), case.k, case.beta, C.c_float(case.tau), acc.data_ptr(), nxt.data_ptr(), z.data_ptr(), name)
    torch.cuda.synchronize()
    assert rc == sd.SPECDEC_OK
    assert np.array_equal(z.cpu().numpy(), out["logits"]) and acc.cpu().tolist() == out["accept"].tolist()
    ses.close()
