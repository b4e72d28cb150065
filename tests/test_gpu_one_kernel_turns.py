"""Who runs passes as one kernel on a GPU: verification keeps it from the first context that asks, and drafting and prefill, which have what verification
leaves, take nothing from it: contexts on two streams, captured passes, another process."""
import contextlib
import ctypes as C
import socket

import numpy as np
import pytest
import torch

import cases
import gpu_harness as gh
import test_gpu_draft_loop as dl
from paper_2203_16487_amd import binding as sd
from paper_2203_16487_amd import synth
from test_gpu_one_kernel import check, desc, resident_launches
from test_gpu_parity_extra import LOGIT_TOL

pytestmark = pytest.mark.gpu
B, K, J, S = 20, 10, 9, 20


@contextlib.contextmanager
def on(stream):
    stream.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(stream):
        yield
        stream.synchronize()


class Drafter:
    """A context with a drafter alone; its passes have 200 drafts of streams of J tokens."""
    def __init__(self, seed=7):
        dd = synth.ModelDesc(1, 2, 512, 8, 2048, 1003, S, 40).resolved()
        self.ses = dl.open_session(B, K, S, 40, dr=(dd, synth.make_weights(dd, seed, tag="drafter", std=0.02)))
        self.toks = synth.random_tokens(seed, "stream", (B, J + 1), dd)
        self.src = synth.random_tokens(seed, "src", (B, S), dd)
        self.dr = torch.zeros((B, K), dtype=torch.int32, device="cuda")
        self.z = torch.zeros((B, K, dd.vocab), dtype=torch.float32, device="cuda")
        self.begin()

    def begin(self):
        sd.specdec_begin(self.ses.ctx, B, 30)
        sd.specdec_encode(self.ses.ctx, self.ses.i32(self.src), self.ses.i32(np.full(B, S)))

    def draft(self):
        """One-kernel launches of a pass, its logits."""
        sd.specdec_set_stream(self.ses.ctx, self.ses.i32(self.toks), self.ses.i32(np.full(B, J)))
        n, _ = resident_launches(self.ses, lambda: sd.specdec_draft(self.ses.ctx, K, self.dr, self.z))
        return n, self.z.cpu().numpy()


def verifier(seed=8):
    case = cases.make_verify_case(desc(512), seed=seed, B=2, S=S, k=5, beta=3, tau=1.0, len_lo=3, len_hi=20, drafts="greedy", ragged_src=True)
    cases.run_oracle(case)
    return case, gh.open_verifier(case, fill=0xFF)


def verified(case, ses):
    """One-kernel launches of a verification pass, which is right."""
    n, out = resident_launches(ses, lambda: gh.gpu_verify(ses, case))
    check(case, out)
    return n


def test_a_drafter_makes_way_for_verification():
    drafter, other = Drafter(), torch.cuda.Stream()
    with on(other):
        n, want = drafter.draft()
        assert n == 1
    case, ses = verifier()
    assert verified(case, ses) == 1
    for end in (False, True):
        if end:
            ses.close()
        with on(other):              # (launches for the rest of the drafter's run)
            n, got = drafter.draft()
            assert n == 0 and np.abs(got - want).max() <= LOGIT_TOL
        if not end:
            assert verified(case, ses) == 1
    with on(other):
        drafter.begin()
        n, got = drafter.draft()
        assert n == 1 and np.array_equal(got, want)
    drafter.ses.close()


def test_on_the_stream_of_verification():
    """In turn with it, and in the same context; on another stream launches, and verification stays."""
    drafter, other = Drafter(), torch.cuda.Stream()
    case, ses = verifier()
    assert verified(case, ses) == 1
    assert drafter.draft()[0] == 1
    sd.specdec_set_stream(ses.ctx, ses.i32(case.tokens), ses.i32(case.lens))
    assert resident_launches(ses, lambda: sd.specdec_prefill(ses.ctx, sd.SPECDEC_VERIFIER))[0] == 1
    assert verified(case, ses) == 1
    with on(other):
        sd.specdec_set_stream(ses.ctx, ses.i32(case.tokens), ses.i32(case.lens))
        assert resident_launches(ses, lambda: sd.specdec_prefill(ses.ctx, sd.SPECDEC_VERIFIER))[0] == 0
    assert verified(case, ses) == 1
    second_case, second = verifier(9)    # (verification's stream is still the first)
    assert verified(second_case, second) == 1
    for s in (ses, second, drafter.ses):
        s.close()


def test_two_drafters():
    one, two, other = Drafter(), Drafter(), torch.cuda.Stream()
    n, want = one.draft()
    assert n == 1
    n, got = two.draft()
    assert n == 1 and np.array_equal(got, want)
    with on(other):
        n, got = two.draft()
        assert n == 0 and np.abs(got - want).max() <= LOGIT_TOL
    one.ses.close()
    two.begin()
    with on(other):
        assert two.draft()[0] == 1
    two.ses.close()


def test_a_captured_draft_leaves_verification_the_gpu():
    drafter, side = Drafter(), torch.cuda.Stream()
    ctx = drafter.ses.ctx
    toks, lens = drafter.ses.i32(drafter.toks), drafter.ses.i32(np.full(B, J))

    def call():
        sd.specdec_set_stream(ctx, toks, lens)
        sd.specdec_draft(ctx, K, drafter.dr, drafter.z)

    graph = torch.cuda.CUDAGraph()
    with on(side):
        sd.specdec_configure(ctx, sd.SPECDEC_OPT_SMALL_BATCH_KERNELS, 0)
        call()
        want = drafter.z.clone()
        sd.specdec_configure(ctx, sd.SPECDEC_OPT_SMALL_BATCH_KERNELS, 1)
        with torch.cuda.graph(graph, stream=side):
            call()
    case, ses = verifier()
    for _ in range(3):
        assert verified(case, ses) == 1
        with on(side):
            drafter.z.zero_()
            graph.replay()
            side.synchronize()
            assert torch.equal(drafter.z, want)
    ses.close()
    drafter.ses.close()


def test_verification_of_another_process():
    """Its lock held by somebody else: launches, until the run after it is given back; a lock that guests hold keeps no verification."""
    path = next(line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64.so" in line)
    bus = C.create_string_buffer(32)
    assert C.CDLL(path).hipDeviceGetPCIBusId(bus, 32, 0) == 0
    drafter = Drafter()

    def hold(name):
        s = socket.socket(socket.AF_UNIX, socket.SOCK_DGRAM)
        s.bind(b"\0" + name + bus.value)
        return s

    with hold(b"specdec-"):
        assert drafter.draft()[0] == 0
    assert drafter.draft()[0] == 0
    drafter.begin()
    assert drafter.draft()[0] == 1
    with hold(b"specdec-"):              # (it comes while drafts have the GPU)
        assert drafter.draft()[0] == 0
    drafter.ses.close()
    with hold(b"specdec-guests-"):
        case, ses = verifier()
        assert verified(case, ses) == 1
        ses.close()
        drafter = Drafter()
        assert drafter.draft()[0] == 0
    drafter.begin()
    assert drafter.draft()[0] == 1
    drafter.ses.close()
