"""What a call's kernels read -- its table of buffers and its plan's tables --
on several streams and under graph capture, on the CPU: the library's host
code over the stand-in of the HIP runtime, which runs work as late as the
calls' own waits allow.  Results against the oracle.
"""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.spawns  # builds the stand-in

BC = synth.BlockCyclic


@pytest.fixture(scope="module")
def standin():
    import standin
    return standin.load()


class Call:
    """One transform (op N, alpha 1, beta 0) with buffers of its own."""

    def __init__(self, S, seed, A, B, layouts=None):
        self.S, self.A, self.B = S, A, B
        self.P = A.nranks
        self.LA, self.LB = layouts or (S.C.layout_from_spec(A), S.C.layout_from_spec(B))
        self.b = [S.array(self.LB.local_elems(r), 1e6 * (seed * self.P + r)) for r in range(self.P)]
        self.a = [S.array(self.LA.local_elems(r), -1.0) for r in range(self.P)]
        self.want = [np.zeros_like(x) for x in self.a]
        oracle.transform("f64", "N", 1.0, 0.0, oracle.OLayout(A), self.want, oracle.OLayout(B), self.b)

    def same_layouts(self, seed):
        return Call(self.S, seed, self.A, self.B, (self.LA, self.LB))

    def run(self, stream, entry="transform"):
        at = lambda bufs: [x.ctypes.data if x.size else None for x in bufs]  # noqa: E731
        if entry == "transform":
            self.S.C.costa_transform("f64", "N", 1.0, 0.0, self.LA, at(self.a), self.LB, at(self.b), stream=stream)
        else:
            d = dict(op="N", alpha=1.0, beta=0.0, A=self.LA, A_local=at(self.a), B=self.LB, B_local=at(self.b))
            self.S.C.costa_transform_batched_noalloc("f64", [d], stream=stream)

    def check(self):
        """The result is there; A is cleared for the next run."""
        self.S.check()
        for x, w in zip(self.a, self.want):
            assert np.array_equal(x, w)
            x[:] = -1.0


def many_ranks(S, seed=0, n=60):
    """128 ranks: a call table of 2160 bytes, more than the kernels' arguments
    hold."""
    return Call(S, seed, BC(64, n, 4, 6, 16, 8, "row", "col"), BC(64, n, 6, 4, 8, 16, "col", "row"))


def test_a_call_waits_for_the_table_that_another_stream_uploads(standin):
    """Two calls of one plan with the same buffers on two streams: the second
    finds its table in the plan's device copy and runs first."""
    S = standin
    c, s1, s2 = many_ranks(S), S.stream(), S.stream()
    c.run(s1)
    c.run(s2)
    S.run(s2)
    c.check()
    # three streams, then other buffers on the first: its table may not
    # overwrite the one that the third stream's call has yet to read
    d, s3 = c.same_layouts(1), S.stream()
    c.run(s1)
    c.run(s2)
    c.run(s3)
    d.run(s1)
    S.run(s1)
    S.run(s3)
    c.check()
    d.check()


def test_a_captured_call_with_a_resident_table_is_accepted(standin):
    """After a call on one stream, the same call is captured on another one,
    replayed, and made uncaptured on a third."""
    S = standin
    c, s1, s2, s3 = many_ranks(S, 2), S.stream(), S.stream(), S.stream()
    c.run(s1)
    S.run(s1)
    c.check()
    S.capture(s2)
    c.run(s2)
    g = S.end_capture(s2)
    for _ in range(2):
        S.replay(g, s1)
        S.run(s1)
        c.check()
    c.run(s3)
    S.run(s3)
    c.check()
    S.destroy_graph(g)


def few_ranks(S, seed=0, m=70, n=90):
    """4 ranks: the call table travels as kernel arguments."""
    return Call(S, seed, BC(m, n, 24, 8, 2, 2, "row", "col"), BC(m, n, 8, 16, 2, 2, "col", "col"))


def test_a_noalloc_call_on_the_null_stream_while_another_stream_captures(standin):
    """hipStreamIsCapturing reports an error for the null stream while a
    blocking stream captures; the call is not part of that capture."""
    S = standin
    c = few_ranks(S)
    S.refuse_implicit(1)
    try:
        c.run(0, "noalloc")
    finally:
        S.refuse_implicit(0)
    S.run(None)
    c.check()


def captured(S, call):
    s = S.stream()
    S.capture(s)
    call.run(s, "noalloc")
    return S.end_capture(s)


def do(S, call, stream, graph=None):
    """Runs the call, or replays its graph, and checks its result alone."""
    if graph is None:
        call.run(stream, "noalloc")
    else:
        S.replay(graph, stream)
    S.run(stream)
    call.check()


@pytest.mark.parametrize("make", [few_ranks, many_ranks], ids=["table_in_arguments", "table_on_device"])
@pytest.mark.parametrize("warm", [False, True])
def test_captured_noalloc_calls_keep_their_buffers(standin, make, warm):
    """Captured and uncaptured calls of one plan with different buffers in any
    order: each replay and each call moves its own."""
    S, s = standin, standin.stream()
    first = make(S, 3, 61 + warm)
    second, third = first.same_layouts(4), first.same_layouts(5)
    if warm:
        do(S, first, s)
    g1 = captured(S, first)
    do(S, first, s)  # the same buffers, before the graph has run
    do(S, second, s)
    do(S, first, s, g1)
    g2 = captured(S, second)
    do(S, first, s, g1)
    do(S, second, s, g2)
    do(S, third, s)
    do(S, second, s, g2)
    do(S, first, s, g1)
    S.destroy_graph(g1)
    do(S, second, s, g2)
    do(S, third, s)
    S.destroy_graph(g2)
    do(S, third, s)
    do(S, first, s)
