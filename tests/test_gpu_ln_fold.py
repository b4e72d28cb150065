"""Precision of LayerNorms folded into the projections around them: sums rounded before their mean is known."""
import numpy as np
import pytest
import torch

import cases
import gpu_harness as gh
from paper_2203_16487_amd import binding as sd
from paper_2203_16487_amd import synth
import specdec_oracle as orc

pytestmark = pytest.mark.gpu


def shifted(desc, seed, shift):
    """A model whose residual sums lie `shift` off zero: a LayerNorm follows every one of them, so this is the same function."""
    bits = synth.make_weights(desc, seed)
    for name in bits:
        if name.endswith((".bo", ".b2")):
            bits[name] = synth.f32_to_bf16_bits(np.full(bits[name].shape, shift, np.float32))
    return bits


def rel(got, want):
    return float(np.linalg.norm(got - want) / np.linalg.norm(want))


def ses_launches(ses, run):
    sd.specdec_profile_select(ses.ctx, sd.KIND["ln"])
    run()
    return sd.specdec_profile_read(ses.ctx)[1]


# Operands are rounded to bf16: with the mean left in, the error of every folded LayerNorm is sqrt(1 + shift^2 / variance) times as
# large, 4 times at shift 4 (sums have standard deviations of 1 .. 1.1).  1.1: errors of two samples of this size.
SHIFT, BOUND = 4.0, 1.1


@pytest.mark.parametrize("d,B,k", [
    (1024, 1, 9), (1024, 9, 8),                     # one kernel over the whole GPU; the last on items of 32 rows
    (512, 1, 25), (512, 12, 10), (512, 30, 10), (1024, 17, 8),   # one kernel, per XCD: the first with weights in place
    (512, 48, 10),                                  # 528 rows: launches
])
def test_verify_of_rows_off_zero(d, B, k):
    desc = synth.ModelDesc(0, 2, d, d // 64, 4 * d, 1003, 64, 64).resolved()
    err = []
    for shift in (0.0, SHIFT):
        case = cases.make_verify_case(desc, seed=3, B=B, S=12, k=k, beta=3, tau=1.0, len_lo=0, len_hi=0)
        case.bits = shifted(desc, 3, shift)
        case.model = orc.Model(desc, synth.weights_f32(case.bits))
        case.states = [orc.new_state(case.model, case.memory[b], k + 1) for b in range(B)]
        cases.run_oracle(case)
        ses = gh.open_verifier(case)
        err.append(rel(gh.gpu_verify(ses, case)["logits"], case.logits))
        ses.close()
    print(f"{d} {B}x{k + 1}: {err[0]:.2e}, off zero {err[1]:.2e}")
    assert err[1] <= BOUND * err[0]


@pytest.mark.parametrize("d,S", [(256, 40), (512, 300)])
def test_encoder_rows_off_zero(d, S):
    desc = synth.ModelDesc(3, 1, d, d // 64, 4 * d, 1003, S, 16).resolved()
    src, err = synth.random_tokens(5, "src", (2, S), desc), []
    for shift, fold in ((0.0, 0), (0.0, 1), (SHIFT, 1)):
        bits = shifted(desc, 5, shift)
        model = orc.Model(desc, synth.weights_f32(bits))
        ses = sd.Session(2, 4, S, 16, fill=0xFF)
        sd.specdec_configure(ses.ctx, sd.SPECDEC_OPT_LN_FOLD, fold)
        ses.bind_model(sd.SPECDEC_VERIFIER, desc, ses.upload_weights(bits))
        sd.specdec_begin(ses.ctx, 2, 8)
        launches = ses_launches(ses, lambda: sd.specdec_encode(ses.ctx, ses.i32(src), ses.i32(np.full(2, S))))
        assert launches == (1 if fold else 2 * desc.enc_layers)        # LayerNorms as launches of their own
        mem = torch.zeros((2, S, d), dtype=torch.bfloat16, device=ses.device)
        sd.specdec_get_memory(ses.ctx, sd.SPECDEC_VERIFIER, mem)
        torch.cuda.synchronize()
        err.append(rel(mem.float().cpu().numpy(), np.stack([orc.encode(model, [int(t) for t in s]) for s in src])))
        ses.close()
    print(f"encoder {d}: not folded {err[0]:.2e}, folded {err[1]:.2e}, off zero {err[2]:.2e}")
    assert max(err[1:]) <= BOUND * err[0]
