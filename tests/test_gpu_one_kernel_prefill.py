"""Prefill passes of few rows (d_model 512) as one kernel, each XCD on sequences of its own, which ends where the last layer's keys and values are
stored: what it caches against the oracle, for streams of different lengths, empty ones among them; waits given up; more rows than it takes."""
import numpy as np
import pytest
import torch

import cases
import gpu_harness as gh
from paper_2203_16487_amd import binding as sd
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
