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


def large_plan(S, seed, rows):
    """About `rows` / 180 MiB of tables (rectangles of one to six elements)."""
    return Call(S, seed, BC(rows, 200, 2, 3, 2, 2, "row", "col"), BC(rows, 200, 3, 2, 2, 2, "col", "col"))


def test_graphs_whose_tables_fill_the_scratch_array(standin):
    """Captured calls hold about 11 of the 16 MiB of tables; calls that find
    no room beside them, captured or not, leave every graph's tables in place,
    and every call finds its own."""
    S, s = standin, standin.stream()
    a, b, c, d = (large_plan(S, 7 + k, 900 + 100 * k) for k in range(4))
    do(S, a, s)
    ga = captured(S, a)  # relies on the tables that the call before it loaded
    gb = captured(S, b)  # holds a copy of its own
    for call in (a, b):
        do(S, call, s, ga if call is a else gb)
    do(S, c, s)          # no room for c, nor for d
    do(S, a, s, ga)
    do(S, c, s)
    do(S, b, s, gb)
    do(S, a, s)
    gd = captured(S, d)
    for _ in range(2):
        do(S, d, s, gd)
        do(S, a, s, ga)
        do(S, c, s)
        do(S, b, s)
        do(S, b, s, gb)
    S.destroy_graph(ga)
    S.destroy_graph(gb)
    do(S, c, s)          # its part may now lie where gd's replays load theirs
    do(S, d, s, gd)
    do(S, c, s)
    gc = captured(S, c)
    do(S, d, s, gd)
    do(S, c, s, gc)
    S.destroy_graph(gd)
    do(S, a, s)
    do(S, c, s, gc)
    S.destroy_graph(gc)
    for call in (a, b, c, d, a):
        do(S, call, s)


def test_graphs_keep_their_plans_past_the_plan_cache_and_finalize(standin):
    """70 other plans start the plan cache over, and costa_finalize drops it:
    a captured call's replays still find their tables."""
    S, s = standin, standin.stream()
    c = few_ranks(S, 11, 50, 60)
    cold = captured(S, c)
    do(S, c, s)
    warm = captured(S, c)
    others = [few_ranks(S, 12, 20, 100 + k) for k in range(70)]
    for o in others:
        do(S, o, s)
    do(S, c, s, warm)
    do(S, c, s, cold)
    S.C.costa_finalize()
    for o in others:
        do(S, o, s)
    do(S, c, s, warm)
    do(S, c, s, cold)
    do(S, c, s)
    S.destroy_graph(cold)
    S.destroy_graph(warm)


@pytest.mark.parametrize("seed", range(6))
def test_captured_and_uncaptured_noalloc_calls_in_random_order(standin, seed):
    S, s = standin, standin.stream()
    rng = np.random.default_rng(seed)
    calls = [large_plan(S, 20 + k, 600 + 250 * k + seed) for k in range(4)] + \
        [many_ranks(S, 30 + k, 70 + 10 * k + seed) for k in range(2)] + [few_ranks(S, 40, 30 + seed)]
    calls += [c.same_layouts(50 + k) for k, c in enumerate(calls[3:])]
    graphs = []
    for _ in range(120):
        what = rng.random()
        if what < 0.2 and len(graphs) < 5:
            k = int(rng.integers(len(calls)))
            graphs.append((calls[k], captured(S, calls[k])))
        elif what < 0.3 and graphs:
            S.destroy_graph(graphs.pop(int(rng.integers(len(graphs))))[1])
        elif what < 0.65 and graphs:
            do(S, graphs[0][0], s, graphs[0][1])
            call, g = graphs[int(rng.integers(len(graphs)))]
            do(S, call, s, g)
        else:
            do(S, calls[int(rng.integers(len(calls)))], s)
    for _, g in graphs:
        S.destroy_graph(g)
