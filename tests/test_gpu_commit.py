"""Commit of a pass: one sequence to more than one round of the block, EOS and caps at every token, failed and finished sequences, against
the rule written out token by token."""
import numpy as np
import pytest
import torch

import cases
import gpu_harness as gh
from paper_2203_16487_amd import binding as sd
from paper_2203_16487_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,k,max_new", [(1, 0, 3), (1, 5, 40), (2, 31, 17), (31, 3, 6), (33, 7, 9), (70, 4, 12), (128, 3, 7), (129, 2, 9), (300, 1, 5)])   # (128 sequences a block)
def test_commit(B, k, max_new):
    desc = synth.ModelDesc(0, 1, 64, 1, 256, 211, 64, 300).resolved()
    case = cases.make_verify_case(desc, seed=B + k, B=B, S=6, k=max(k, 1), beta=3, tau=1.0, len_lo=0, len_hi=9, drafts="random", ragged_src=True)
    ses = sd.Session(B, max(k, 1), 6, 80)
    ses.bind_model(sd.SPECDEC_VERIFIER, desc, ses.upload_weights(case.bits))
    sd.specdec_begin(ses.ctx, B, max_new)
    sd.specdec_set_memory(ses.ctx, sd.SPECDEC_VERIFIER, ses.bf16(case.memory), ses.i32(case.src_len))
    sd.specdec_set_stream(ses.ctx, ses.i32(case.tokens), ses.i32(case.lens))
    sd.specdec_prefill(ses.ctx, sd.SPECDEC_VERIFIER)
    rng = np.random.default_rng([B, k])
    out, done, total = [[] for _ in range(B)], [False] * B, 0
    acc, nxt = ses.i32(np.zeros(B)), ses.i32(np.zeros(B))
    toks, n, fin, active, cnt = (torch.zeros(s, dtype=torch.int32, device="cuda") for s in ((B, 64), B, B, 1, sd.SPECDEC_COUNTERS))
    for turn in range(1, 5):
        drafts = rng.integers(4, 210, size=(B, max(k, 1)))
        drafts[rng.random(drafts.shape) < 0.1] = desc.eos_id
        sd.specdec_verify(ses.ctx, ses.i32(drafts) if k else None, k, 1, 0.0, acc, nxt)
        a = rng.integers(0, k + 3, size=B)                  # (beyond k: k)
        a[rng.random(B) < 0.1] = -1
        last = rng.integers(4, 210, size=B)
        last[rng.random(B) < 0.1] = desc.eos_id
        sd.specdec_commit(ses.ctx, ses.i32(a), ses.i32(last), active)
        sd.specdec_get_output(ses.ctx, toks, n, fin)
        sd.specdec_get_counters(ses.ctx, cnt)
        for b in range(B):
            if done[b] or a[b] < 0:
                continue
            m = min(int(a[b]), k)
            for t in [int(x) for x in drafts[b, :m]] + [int(last[b])]:
                out[b].append(t)
                total += 1
                if t == desc.eos_id or len(out[b]) == max_new:
                    done[b] = True
                    break
        assert n.cpu().tolist() == [len(o) for o in out] and fin.cpu().tolist() == [int(x) for x in done]
        for b in range(B):
            assert toks[b, :len(out[b])].cpu().tolist() == out[b], b
        assert int(active) == B - sum(done) and cnt[:3].cpu().tolist() == [turn, total, sum(done)]
    ses.close()
