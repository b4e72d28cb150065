"""The work a serving program has this library do, as measurable cases: one pass each through the public entry points of
`paper_2203_16487_amd.binding`.

A case is a dict of plain values.  `kind` says which calls a pass makes:

  verify   one verification pass of the drafts in hand and its row statistics (the log-probabilities a service returns)
  step     one step of plain autoregressive decoding: verify with k = 0, commit (and rewind, so that passes repeat)
  loop     one iteration of the draft-then-verify loop: verify, statistics, commit, draft, statistics (and rewind)
  draft    a drafter resumed from a stored prefix (streams + keys / values) drafts the next k tokens
  resume   decoding resumed from tokens alone: set the streams, prefill the verifier, verify the drafts in hand
  encode   a new batch of sources: begin, encode with every model, first token of every sequence, memories read back

`verifier` / `drafter` name the model shapes of the paper's setups ("" = not bound): "base" 6 layers 512 / 2048, "big" 6 layers
1024 / 4096, "deep-shallow" 12 + 2 layers 512 / 2048.  Prefix lengths are uniform in [j_lo, j_hi], source lengths in [s_lo, s_hi].

Inputs.  Weights are N(0, 0.02) like everywhere in this repository, except that the matrices which end a residual branch are half
that (trained branches are small next to the stream they add to).  With the tied output matrix the verifier then favours the token
it has just read by a clear margin, as a trained model favours its continuation by a clear margin: a draft that repeats the pending
token is accepted, a random one is not, and neither decision hangs on the last bit of a sum.  Drafts repeat the pending token
with every position replaced by a random token at probability 0.2.  The [MASK] row is a tenth of a token's, so that the slots of an
untrained drafter do not all predict [MASK]."""
import numpy as np
import torch

from paper_2203_16487_amd import binding as sd
from paper_2203_16487_amd import synth

V32K = 32768


def listed():
    def case(name, kind, verifier, drafter, B, k, s, j, **more):
        return dict(dict(name=name, kind=kind, verifier=verifier, drafter=drafter, B=B, k=k, s_lo=s[0], s_hi=s[1], j_lo=j[0], j_hi=j[1],
                         vocab=V32K, beta=3, tau=1.0, fp8_weights=False, fp8_cross_kv=False), **more)

    return [
        # one user waiting for one sentence: the smallest pass there is, bound by launches and latency
        case("verify one, base, k=5", "verify", "base", "", 1, 5, (32, 32), (16, 16)),
        # the same with the big model at the paper's best block size, weights stored in 8 bits to halve what is streamed
        case("verify one, big, k=25, fp8 weights", "verify", "big", "", 1, 25, (90, 90), (57, 57), fp8_weights=True),
        # a handful of users at once: more rows than the small-batch kernels take, far fewer than fill the chip; odd sizes
        case("verify 7, base, k=10, ragged", "verify", "base", "", 7, 10, (9, 61), (0, 75), vocab=32003),
        # a batched translation service on the base model (the batched verify step of the workload definitions)
        case("verify 32, base, k=10", "verify", "base", "", 32, 10, (64, 64), (0, 64)),
        # summarization: long sources, cross-attention streams most of the bytes
        case("verify 32, big, source 1024", "verify", "big", "", 32, 10, (1024, 1024), (200, 245), beta=5, tau=3.0),
        # the same work with 8-bit cross keys / values, a ragged batch and an odd vocabulary
        case("verify 19, big, ragged, fp8 cross", "verify", "big", "", 19, 10, (333, 777), (11, 190), vocab=32003, beta=5, tau=3.0,
             fp8_cross_kv=True),
        # the autoregressive baseline at full batch: one row per sequence
        case("step 128, big", "step", "big", "", 128, 0, (16, 128), (48, 64)),
        # the translation loop at full batch, the repository's headline workload
        case("loop 128, big + drafter", "loop", "big", "deep-shallow", 128, 10, (16, 128), (48, 64)),
        # the drafter's pass on its own
        case("draft 64", "draft", "", "deep-shallow", 64, 10, (128, 128), (32, 32)),
        # requests that come back with their text but without their cache
        case("resume 32, big, 224 tokens", "resume", "big", "", 32, 10, (128, 512), (130, 224)),
        # a new batch of sentences, and a new batch of articles
        case("encode 128 sentences", "encode", "big", "deep-shallow", 128, 10, (16, 128), (0, 0)),
        case("encode 32 articles", "encode", "big", "deep-shallow", 32, 10, (1024, 1024), (0, 0)),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(lo * (hi / lo) ** rng.random()))))


def draw(rng):
    kind = rng.choice(["verify", "verify", "verify", "step", "loop", "draft", "resume", "encode"])
    verifier = "" if kind == "draft" else rng.choice(["base", "big"])
    drafter = "deep-shallow" if kind in ("loop", "draft", "encode") else ""
    k = 0 if kind == "step" else rng.choice([5, 7, 10, 10, 15, 20, 25])
    rows = _log_int(rng, k + 1, 1408)          # rows of a pass: a single sequence .. the full batch
    B = max(1, min(128, rows // (k + 1)))
    j_hi = _log_int(rng, 4, 245)
    s_hi = _log_int(rng, 8, 1024)
    if kind == "encode":
        j_hi, B = 0, max(1, min(128, _log_int(rng, s_hi, 32768) // s_hi))
    else:
        s_hi = min(s_hi, 32768 // B)           # key rows of a batch: the largest listed has 32 x 1024
    j_lo = rng.choice([j_hi, j_hi // 2, 0])
    s_lo = rng.choice([s_hi, max(1, s_hi // 2), max(1, s_hi // 8)])
    return dict(kind=kind, verifier=verifier, drafter=drafter, B=B, k=k, s_lo=s_lo, s_hi=s_hi, j_lo=j_lo, j_hi=j_hi,
                vocab=rng.choice([V32K, V32K, rng.randrange(30000, 34000)]), beta=rng.choice([1, 3, 5]), tau=rng.choice([1.0, 3.0]),
                fp8_weights=kind == "verify" and rng.random() < 0.2, fp8_cross_kv=kind != "draft" and rng.random() < 0.2)


def _desc(case, which):
    enc = case["kind"] == "encode"
    if which == "deep-shallow":
        return synth.spec_drafter(enc_layers=12 if enc else 0, vocab=case["vocab"])
    return (synth.big_verifier if which == "big" else synth.base_verifier)(enc_layers=6 if enc else 0, vocab=case["vocab"])


def _weights(desc, gen):
    out = []
    for name, shape, what in synth.tensor_specs(desc):
        std = 0.01 if name.endswith((".wo", ".w2")) else 0.02
        w = torch.randn(shape, generator=gen, device="cuda") * std
        if what == "g":
            w += 1.0
        if name == "embed":
            w[desc.mask_id] *= 0.1
        out.append(w.to(torch.bfloat16))
    return out


def prepare(case, seed):
    """Models bound, memories set, streams and caches in place: a server between two calls."""
    B, k, kind = case["B"], case["k"], case["kind"]
    gen = torch.Generator(device="cuda").manual_seed(seed)
    rng = np.random.default_rng([seed, 1])
    k_max = max(k, 10)
    max_tgt = 128 if case["j_hi"] <= 96 else 256
    ses = sd.Session(B, k_max, case["s_hi"], max_tgt)
    sd.specdec_configure(ses.ctx, sd.SPECDEC_OPT_FP8_WEIGHTS, int(case["fp8_weights"]))
    sd.specdec_configure(ses.ctx, sd.SPECDEC_OPT_FP8_CROSS_KV, int(case["fp8_cross_kv"]))
    roles = [(sd.SPECDEC_VERIFIER, case["verifier"]), (sd.SPECDEC_DRAFTER, case["drafter"])]
    roles = [(role, _desc(case, which)) for role, which in roles if which]
    desc = roles[0][1]
    for role, dsc in roles:
        ses.bind_model(role, dsc, _weights(dsc, gen))

    def ints(lo, hi, shape):
        return rng.integers(lo, hi + 1, size=shape, dtype=np.int64).astype(np.int32)

    def zeros(*shape, dtype=torch.int32):
        return torch.zeros(shape, dtype=dtype, device="cuda")

    st = dict(case=case, ses=ses, ctx=ses.ctx, k=k, acc=zeros(B), nxt=zeros(B), nact=zeros(1))
    s_len = ints(case["s_lo"], case["s_hi"], B)
    s_len[0] = case["s_hi"]
    st["s_len"] = ses.i32(s_len)
    st["stats"] = zeros(B, 1 if kind == "encode" else k + 1, sd.SPECDEC_ROW_STATS, dtype=torch.float32)
    # the columns a service reads (next_token carries the arg-max of the row that counts)
    st["scores"] = {"max": st["stats"][..., 0], "lse": st["stats"][..., 2], "draft": st["stats"][..., 3], "above": st["stats"][..., 4]}
    if kind == "encode":
        st["src"] = ses.i32(ints(4, desc.vocab - 2, (B, case["s_hi"])))
        st["mem"] = [(role, zeros(B, case["s_hi"], d.d_model, dtype=torch.bfloat16)) for role, d in roles]
        return st
    sd.specdec_begin(ses.ctx, B, 10 ** 6)
    for role, d in roles:
        mem = torch.randn((B, case["s_hi"], d.d_model), generator=gen, device="cuda").to(torch.bfloat16)
        sd.specdec_set_memory(ses.ctx, role, mem, st["s_len"])
    lens = ints(case["j_lo"], case["j_hi"], B)
    lens[0] = case["j_hi"]
    toks = ints(4, desc.vocab - 2, (B, case["j_hi"] + 1))
    toks[:, 0] = desc.bos_id
    pending = toks[np.arange(B), lens]
    drafts = np.where(rng.random((B, max(k, 1))) < 0.2, ints(0, desc.vocab - 1, (B, max(k, 1))), pending[:, None])
    st.update(toks=ses.i32(toks), lens=ses.i32(lens), drafts=ses.i32(drafts), zero=zeros(B))
    sd.specdec_set_stream(ses.ctx, st["toks"], st["lens"])
    for role, d in roles:
        sd.specdec_prefill(ses.ctx, role)
    if drafted := [d for role, d in roles if role == sd.SPECDEC_DRAFTER]:
        st["out"] = zeros(B, k)
        st["dstats"] = zeros(B, k, sd.SPECDEC_ROW_STATS, dtype=torch.float32)
        st["dmax"] = st["dstats"][..., 0]
        if kind == "draft":
            shape = (drafted[0].dec_layers, B, case["j_hi"], drafted[0].d_model)
            st["kc"], st["vc"] = zeros(*shape, dtype=torch.bfloat16), zeros(*shape, dtype=torch.bfloat16)
            sd.specdec_get_cache(ses.ctx, sd.SPECDEC_DRAFTER, st["kc"], st["vc"])
    return st


def run(st):
    case, ctx, k = st["case"], st["ctx"], st["k"]
    kind, acc, nxt = case["kind"], st["acc"], st["nxt"]
    if kind == "draft":
        sd.specdec_set_prefix(ctx, sd.SPECDEC_DRAFTER, st["toks"], st["lens"], st["kc"], st["vc"])
        sd.specdec_draft(ctx, k, st["out"])
        sd.specdec_get_draft_stats(ctx, st["dstats"])
        return {"draft": st["out"], "max": st["dmax"]}
    if kind == "encode":
        sd.specdec_begin(ctx, case["B"], 10 ** 6)
        sd.specdec_encode(ctx, st["src"], st["s_len"])
        for role, mem in st["mem"]:
            sd.specdec_get_memory(ctx, role, mem)
        sd.specdec_verify(ctx, None, 0, 1, 0.0, acc, nxt)
        sd.specdec_get_row_stats(ctx, st["stats"])
        return {"next": nxt, "max": st["scores"]["max"], "lse": st["scores"]["lse"], "memory": [mem for _, mem in st["mem"]]}
    if kind == "step":
        sd.specdec_verify(ctx, None, 0, 1, 0.0, acc, nxt)
        sd.specdec_get_row_stats(ctx, st["stats"])
        sd.specdec_commit(ctx, st["zero"], nxt, st["nact"])
        sd.specdec_rewind(ctx, st["lens"])
        return {"next": nxt, "active": st["nact"], "max": st["scores"]["max"], "lse": st["scores"]["lse"]}
    if kind == "resume":
        sd.specdec_set_stream(ctx, st["toks"], st["lens"])
        sd.specdec_prefill(ctx, sd.SPECDEC_VERIFIER)
    sd.specdec_verify(ctx, st["drafts"], k, case["beta"], case["tau"], acc, nxt)
    sd.specdec_get_row_stats(ctx, st["stats"])
    got = {"accept": acc, "next": nxt, "scores": st["scores"]}
    if kind == "loop":
        sd.specdec_commit(ctx, acc, nxt, st["nact"])
        sd.specdec_draft(ctx, k, st["out"])
        sd.specdec_get_draft_stats(ctx, st["dstats"])
        sd.specdec_rewind(ctx, st["lens"])
        got.update(active=st["nact"], draft=st["out"], draft_max=st["dmax"])
    return got


def _decoder_pass(case, which, rows, vocab_rows, keys):
    """Bytes and operations of one decoder pass: matrices once, cached keys / values once, new ones written once."""
    d = _desc(case, which)
    D, F, V, L, B = d.d_model, d.d_ffn, d.vocab, d.dec_layers, case["B"]
    per_weight = 1 if case["fp8_weights"] and rows <= 32 else 2
    s = (case["s_lo"] + case["s_hi"]) / 2
    cross = (1 + 4 / 64) if case["fp8_cross_kv"] else 2
    nbytes = per_weight * (L * (6 * D * D + 2 * D * F) + (V * D if vocab_rows else 0))
    nbytes += L * 2 * D * B * (2 * keys + cross * s) + 2 * D * rows
    flops = 2.0 * rows * L * (6 * D * D + 2 * D * F) + 2.0 * vocab_rows * V * D + 4.0 * rows * L * D * (keys + s)
    return nbytes, flops


def work(case):
    B, k, kind = case["B"], case["k"], case["kind"]
    s, j = (case["s_lo"] + case["s_hi"]) / 2, (case["j_lo"] + case["j_hi"]) / 2
    parts = []
    if kind == "encode":
        for which in (case["verifier"], case["drafter"]):
            d = _desc(case, which)
            D, F, n = d.d_model, d.d_ffn, B * s
            square = B * (case["s_lo"] ** 2 + case["s_lo"] * case["s_hi"] + case["s_hi"] ** 2) / 3   # mean of S^2
            cross = (1 + 4 / 64) if case["fp8_cross_kv"] else 2
            parts.append((2 * (d.enc_layers * (4 * D * D + 2 * D * F) + d.dec_layers * 2 * D * D) + n * D * 2 * 2 +
                          d.dec_layers * 2 * D * n * cross,
                          2.0 * n * (d.enc_layers * (4 * D * D + 2 * D * F) + d.dec_layers * 2 * D * D) + 4.0 * d.enc_layers * D * square))
        parts.append(_decoder_pass(case, case["verifier"], B, B, 1))
    if kind in ("verify", "step", "loop", "resume"):
        parts.append(_decoder_pass(case, case["verifier"], B * (k + 1), B * (k + 1), j + k + 1))
    if kind == "resume":   # the prefix itself: every position's rows once, half the prefix visible on average
        D = _desc(case, case["verifier"])
        flops = 2.0 * B * j * D.dec_layers * (6 * D.d_model ** 2 + 2 * D.d_model * D.d_ffn) + 4.0 * B * j * D.dec_layers * D.d_model * (j / 2 + s)
        parts.append((2 * D.dec_layers * 2 * D.d_model * B * j, flops))
    if kind in ("loop", "draft"):
        fresh = B if kind == "draft" else B * (1 + k / 3)   # stream rows ingested beside the mask slots
        parts.append(_decoder_pass(case, case["drafter"], fresh + B * k, B * k, j + 1 + k))
    if kind == "draft":    # the stored prefix is read
        D = _desc(case, case["drafter"])
        parts.append((2 * D.dec_layers * 2 * D.d_model * B * j, 0.0))
    return {"bytes": float(sum(p[0] for p in parts)), "flops": float(sum(p[1] for p in parts))}


def tolerance(case):
    # bf16 operands (or 8-bit ones re-read as bf16) with fp32 sums: logits, statistics and memories to about 1e-2; a token may
    # differ only where two logits lie closer than that
    return {"rel": 1e-2, "differ": 0.01}
