"""Passes of at most 63 rows at d_model 512 on the per-XCD decoder, which then reads the matrices as they are bound: one and two row tiles of
a group, groups with a sequence more than others, fewer groups than XCDs; and on a stream with half of the compute units, where the
decoder over the whole GPU or separate launches take them."""
import numpy as np
import pytest
import torch

import cases
import gpu_harness as gh
from paper_2203_16487_amd import binding as sd
from test_gpu_one_kernel import FP8_KV, check, desc, masked_stream, resident_launches

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,k,S,lo,hi,opts,half", [
    (1, 0, 9, 0, 0, {}, 1),              # one row, nothing cached; (half: launches of the one-kernel decoder on half of the compute units)
    (1, 15, 40, 31, 33, {}, 1),          # 16 rows: one whole row tile
    (1, 31, 50, 60, 64, {}, None),       # 32: two, two query tiles
    (3, 20, 70, 0, 90, {}, None),        # 21 on three XCDs
    (8, 6, 64, 48, 64, FP8_KV, 0),       # 7 on each
    (9, 6, 64, 0, 64, {}, 0),            # 14 on one, 7 on the others
    (60, 0, 20, 0, 40, {}, None),        # 8 and 7
])
def test_few_rows_in_place(B, k, S, lo, hi, opts, half):
    case = cases.make_verify_case(desc(512, 3), seed=600 + 10 * B + k, B=B, S=S, k=k, beta=3, tau=1.0, len_lo=lo, len_hi=hi, drafts="random",
                                  ragged_src=True, fp8_kv=sd.SPECDEC_OPT_FP8_CROSS_KV in opts)
    cases.run_oracle(case)
    ses = gh.open_verifier(case, k_max=max(k, 1), options=opts, fill=0xFF)
    n, out = resident_launches(ses, lambda: gh.gpu_verify(ses, case))
    assert n == 1 and sd.specdec_decoder_way(ses.ctx) == "xcd in place"
    check(case, out)
    assert np.array_equal(gh.gpu_verify(ses, case)["logits"], out["logits"])
    K, V = gh.gpu_cache(ses, case, case.L_max + k + 1)
    for b, st in enumerate(case.states):
        j = int(case.lens[b])
        for l in range(case.desc.dec_layers):
            assert np.abs(K[l, b, j:j + k + 1] - st.K[l][j:j + k + 1]).max() <= 3e-2, (b, l)
            assert np.abs(V[l, b, j:j + k + 1] - st.V[l][j:j + k + 1]).max() <= 3e-2, (b, l)
    if half is not None:
        torch.cuda.synchronize()
        stream = masked_stream([0xffffffff] * 4 + [0] * 4)
        with torch.cuda.stream(stream):
            n, apart = resident_launches(ses, lambda: gh.gpu_verify(ses, case))
        stream.synchronize()
        assert n == half and sd.specdec_decoder_way(ses.ctx) == ("gpu" if half else "launches")
        check(case, apart)
    ses.close()
