"""Passes of more than 64 rows to an XCD (d_model 512: up to 160, 1024: up to 96): verification and drafting as one kernel, five to ten row
tiles and their remainders, summed all at once and a few at a time, against the oracle; waits given up; more rows than it takes."""
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


@pytest.mark.parametrize("way,d,B,k,S,lo,hi,opts", [
    ("xcd in place", 512, 34, 12, 20, 0, 40, {}),       # 65 and 52 rows, five tiles: the last of one row
    ("xcd in place", 512, 40, 15, 30, 0, 60, FP8_KV),   # 80, five
    ("xcd in place", 512, 64, 10, 64, 0, 64, {}),       # 88, six
    ("xcd in place", 512, 43, 15, 300, 0, 200, {}),     # 96 and 80, six; several chunks of keys
    ("xcd in place", 512, 97, 7, 30, 0, 75, FP8_KV),    # 104 and 96, seven
    ("xcd in place", 512, 32, 27, 20, 0, 40, {}),  # 112, seven; two query tiles a sequence
    ("xcd in place", 512, 81, 10, 20, 0, 40, {}),  # 121 and 110, eight
    ("xcd in place", 512, 43, 21, 20, 0, 40, FP8_KV),   # 132 and 110, nine
    ("xcd in place", 512, 112, 10, 64, 0, 64, {}), # 154, ten
    ("xcd in place", 512, 80, 15, 20, 0, 40, {}),  # 160, ten: 1280 rows, the most
    ("launches", 512, 121, 10, 20, 0, 40, {}),     # 176 and 165
    ("xcd", 1024, 34, 12, 20, 0, 40, {}),          # 65 and 52, five
    ("xcd", 1024, 40, 15, 200, 0, 140, FP8_KV),    # 80, five
    ("xcd", 1024, 64, 10, 40, 0, 64, {}),          # 88, six
    ("xcd", 1024, 24, 31, 40, 0, 64, {}),          # 96, six: 768 rows, the most; two query tiles a sequence
    ("launches", 1024, 33, 21, 20, 0, 40, {}),     # 110 and 88
])
def test_verification_against_oracle(way, d, B, k, S, lo, hi, opts):
    case = cases.make_verify_case(desc(d), seed=600 + B, B=B, S=S, k=k, beta=3, tau=1.0, len_lo=lo, len_hi=hi, drafts="random", ragged_src=True,
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
    (41, 10, 20, (0, 10), False),       # up to 126 and 105, eight
    (97, 10, 20, (0, 30), True),        # 143 and 132, nine: the most
])
def test_drafting_against_oracle(B, k, S, j, prefill):
    dd, db, dm = model()
    lens = synth.random_lengths(700 + B, "len", B, *j)
    lens[0] = j[1]
    px.drafter_pass_case(dd, db, dm, B=B, S_max=S, k=k, lens=lens, seed=700 + B, prefill=prefill, max_tgt=330, sample=(0, B // 2, B - 1), one=1)


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
