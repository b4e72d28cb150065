"""Passes of 65 - 112 rows to an XCD (d_model 512): verification and drafting as one kernel, five to seven row tiles and their remainders,
against the oracle; waits given up; one row more than it takes."""
import numpy as np
import pytest

import cases
import gpu_harness as gh
import test_gpu_parity_extra as px
from paper_2203_16487_amd import binding as sd
from paper_2203_16487_amd import synth
from test_gpu_one_kernel import FP8_KV, check, desc, resident_launches
from test_gpu_one_kernel_draft import draft, model, open_pass

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("way,B,k,S,lo,hi,opts", [
    ("xcd in place", 34, 12, 20, 0, 40, {}),       # 65 and 52 rows, five tiles: the last of one row
    ("xcd in place", 40, 15, 30, 0, 60, FP8_KV),   # 80, five
    ("xcd in place", 64, 10, 64, 0, 64, {}),       # 88, six
    ("xcd in place", 43, 15, 300, 0, 200, {}),     # 96 and 80, six; several chunks of keys
    ("xcd in place", 97, 7, 30, 0, 75, FP8_KV),    # 104 and 96, seven
    ("xcd in place", 32, 27, 20, 0, 40, {}),       # 112, seven: 896 rows, the most; two query tiles a sequence
    ("launches", 33, 27, 20, 0, 40, {}),           # 140 and 112
])
def test_verification_against_oracle(way, B, k, S, lo, hi, opts):
    case = cases.make_verify_case(desc(512), seed=600 + B, B=B, S=S, k=k, beta=3, tau=1.0, len_lo=lo, len_hi=hi, drafts="random", ragged_src=True,
                                  fp8_kv=sd.SPECDEC_OPT_FP8_CROSS_KV in opts)
    cases.run_oracle(case)
    ses = gh.open_verifier(case, k_max=k, options=opts, fill=0xFF)
    out = gh.gpu_verify(ses, case)
    assert sd.specdec_decoder_way(ses.ctx) == way
    K, V = gh.gpu_cache(ses, case, case.L_max + k + 1)
    check(case, out)
    for give_up in (1, 0):
        sd.specdec_configure(ses.ctx, sd.SPECDEC_OPT_GIVE_UP_WAITS, give_up)
        got = gh.gpu_verify(ses, case)
        for key in ("logits", "accept", "next", "stats"):
            assert np.array_equal(got[key], out[key]), (give_up, key)
    ses.close()
    for b, st in enumerate(case.states):
        j = int(case.lens[b])
        for l in range(case.desc.dec_layers):
            assert np.abs(K[l, b, j:j + k + 1] - st.K[l][j:j + k + 1]).max() <= 3e-2, (b, l)
            assert np.abs(V[l, b, j:j + k + 1] - st.V[l][j:j + k + 1]).max() <= 3e-2, (b, l)


@pytest.mark.parametrize("B,k,S,j,prefill", [
    (64, 10, 40, (0, 40), True),        # 88 places, six tiles
    (16, 25, 30, (0, 25), False),       # up to 102, seven; half of them without rows
    (40, 7, 20, (0, 7), False),         # up to 75, five
    (33, 15, 260, (200, 290), True),    # 80 and 64, five
])
def test_drafting_against_oracle(B, k, S, j, prefill):
    dd, db, dm = model()
    lens = synth.random_lengths(700 + B, "len", B, *j)
    lens[0] = j[1]
    px.drafter_pass_case(dd, db, dm, B=B, S_max=S, k=k, lens=lens, seed=700 + B, prefill=prefill, max_tgt=330, sample=(0, B // 2, B - 1))


def test_drafting_given_up():
    B, k = 64, 10
    ses, dd, toks, lens = open_pass(B, k, (20, 40), 701)
    sd.specdec_prefill(ses.ctx, sd.SPECDEC_DRAFTER)
    n, _ = resident_launches(ses, lambda: draft(ses, dd, B, k, lens, False))
    assert n == 1
    want = draft(ses, dd, B, k, lens, True)
    for give_up in (1, 0):
        sd.specdec_configure(ses.ctx, sd.SPECDEC_OPT_GIVE_UP_WAITS, give_up)
        got = draft(ses, dd, B, k, lens, True)
        assert np.array_equal(got[1], want[1]) and np.array_equal(got[0], want[0]), give_up
    ses.close()
