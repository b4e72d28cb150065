"""FFN2 + sum of d_model 1024 on tiles of 96 x 64 whose waves' rings take all of the LDS (1025 - 1536 rows): remainders of the last row tile, the
smallest and the largest pass; against the oracle."""
import numpy as np
import pytest

import cases
import gpu_harness as gh
from test_gpu_one_kernel import check, desc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,k,hi", [
    (41, 24, 40),       # 1025 rows: 65 in the last tile
    (53, 23, 40),       # 1272: 24
    (128, 10, 64),      # 1408: 64
    (128, 11, 30),      # 1536: whole tiles
])
def test_verification_against_oracle(B, k, hi):
    case = cases.make_verify_case(desc(1024), seed=800 + B + k, B=B, S=20, k=k, beta=3, tau=1.0, len_lo=0, len_hi=hi, drafts="random", ragged_src=True)
    cases.run_oracle(case)
    ses = gh.open_verifier(case, k_max=k, fill=0xFF)
    out = gh.gpu_verify(ses, case)
    K, V = gh.gpu_cache(ses, case, case.L_max + k + 1)
    check(case, out)
    got = gh.gpu_verify(ses, case)
    ses.close()
    for key in ("logits", "accept", "next", "stats"):
        assert np.array_equal(got[key], out[key]), key
    for b, st in enumerate(case.states):
        j = int(case.lens[b])
        for l in range(case.desc.dec_layers):
            assert np.abs(K[l, b, j:j + k + 1] - st.K[l][j:j + k + 1]).max() <= 3e-2, (b, l)
            assert np.abs(V[l, b, j:j + k + 1] - st.V[l][j:j + k + 1]).max() <= 3e-2, (b, l)
