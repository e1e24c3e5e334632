"""Batched calls recorded into a graph of the caller's: other batched calls go on
while the capture is open, and the graph stays good after other calls have gone
through the cache of schedules.  Outputs equal the single calls' bit for bit."""
import numpy as np
import pytest
import torch

from paper_2303_08879_amd import fockdiag as F
from paper_2303_08879_amd import ops
from paper_2303_08879_amd import workloads as W

pytestmark = pytest.mark.gpu
DT = torch.complex128


class Call:
    """Plans, inputs and buffers of a batch: both algorithms, so that several
    classes of launches stand side by side."""

    def __init__(self):
        self.circs = [W.config1(), W.config2(c_u=6, c_d=4), W.config5(c=2)]
        self.plans = [F.Plan(c.cutoffs, c.detected_mask, DT, "general") for c in self.circs]
        self.ins = [ops._as_inputs(c.A, c.b, c.c, DT, "cuda") for c in self.circs]
        self.ws = [ops._workspace(p.workspace(False)[0], "cuda") for p in self.plans]
        self.rho = self.outputs()
        self.ref = [ops.fock_diag(c.A, c.b, c.c, c.cutoffs, c.detected_mask, DT, "general") for c in self.circs]

    def outputs(self):
        return [torch.zeros(p.out_shape, dtype=DT, device="cuda") for p in self.plans]

    def run(self, rho=None):
        F.fock_diag_fwd_batch(self.plans, [x[0] for x in self.ins], [x[1] for x in self.ins],
                              [x[2] for x in self.ins], rho or self.rho, self.ws)

    def check(self):
        torch.cuda.synchronize()
        for r, x in zip(self.rho, self.ref):
            assert torch.equal(r, x)
            r.zero_()


@pytest.fixture
def eager_batches():
    old = F.fd_batch_get_tuning()
    F.fd_batch_set_tuning(*old[:4], 0)
    yield
    F.fd_batch_set_tuning(*old[:4], max(old[4], 0))


def capture(call, during=None):
    s1 = torch.cuda.Stream()
    with torch.cuda.stream(s1):
        call.run()                  # the schedule's tables
    call.check()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=s1, capture_error_mode="thread_local"):
        call.run()
        if during is not None:
            during()
    return graph


def test_other_calls_while_a_capture_is_open(eager_batches):
    a, b = Call(), Call()
    b.run()
    b.check()
    s2 = torch.cuda.Stream()

    def other():
        with torch.cuda.stream(s2):
            b.run()

    print("[batch capture] a batched call on another stream inside the capture", flush=True)
    graph = capture(a, other)
    b.check()
    for _ in range(3):
        graph.replay()
        b.run()
        a.check()
        b.check()


def test_captured_call_outlives_the_cache(eager_batches):
    a, b = Call(), Call()
    print("[batch capture] replay after twelve other schedules", flush=True)
    graph = capture(a)
    for _ in range(12):
        b.run(b.outputs())
    torch.cuda.synchronize()
    for _ in range(3):
        graph.replay()
        a.check()
        b.run()
        b.check()
