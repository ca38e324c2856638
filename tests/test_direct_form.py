"""The direct form of a transform against its message form and the oracle.

CPU: the direct form's rectangles, applied on host buffers as the kernels
address them, stay in bounds, write every element of A once and reproduce the
oracle bit for bit, over orders, types, ops, ragged and windowed layouts.
GPU: both forms give the same bits; calls whose A and B buffers share memory
take the message form and give what it gives.
"""
import numpy as np
import pytest
import torch

import oracle
import synth
from replay import _combine, _index, many_rank_cases, random_stack_case, short_walk_cases, stack_cases
from test_plan_replay import CAP, DIRECT, MAXX, _descs, _written_mask, check_tasks, stack_walk_cover

C = pytest.importorskip("paper_2106_06601_amd")
BC, GEN, SL = synth.BlockCyclic, synth.General, synth.ScaLapack


# elements and width of the tiles that one wave moves (launches of small tiles)
SMALL, SMALL_X = {4: 1024, 8: 768, 16: 512}, 64
BUDGET = {4: 4096, 8: 2048, 16: 3072}  # of 256-lane tiles


def check_tiles(ps, es):
    """A launch of tiles: workgroups numbered in rectangle order, one per
    tile, and every tile within the limits (elements, width, LDS array) of the
    launch's workgroups, of one wave or of 256 lanes."""
    lanes = int(ps[0]["reserved"])
    assert lanes in (64, 256)
    budget, lds, maxx = (SMALL[es], SMALL[es] + SMALL_X, SMALL_X) if lanes == 64 else (BUDGET[es], CAP[es], MAXX[es])
    nxt = 0
    for p in ps:
        nx, ny, x, y = int(p["nx"]), int(p["ny"]), int(p["tile_x"]), int(p["tile_y"])
        assert int(p["flags"]) & 1 and 1 <= x <= nx and 1 <= y <= ny and int(p["reserved"]) == lanes
        assert x <= maxx and x * y <= budget and x * (y | 1) <= lds
        assert int(p["group"]) == nxt and int(p["ntasks"]) == -(-nx // x) * -(-ny // y)
        nxt += int(p["ntasks"])
    return lanes


def _random_workload(seed):
    """Random layouts: all four types, ops, orders and scalar modes by seed."""
    rng = np.random.default_rng(seed)
    P = int(rng.integers(1, 7))
    M, N = int(rng.integers(1, 150)), int(rng.integers(1, 150))
    op = "NTC"[seed % 3]
    dtype = ["f64", "c128", "f32", "c64"][seed % 4]

    def lay(m, n):
        order = "col" if rng.random() < 0.5 else "row"
        if rng.random() < 0.5:
            return BC(m, n, int(rng.integers(1, 40)), int(rng.integers(1, 40)), 1, P,
                      "row" if rng.random() < 0.5 else "col", order)
        nr, nc = int(rng.integers(1, min(m, 6) + 1)), int(rng.integers(1, min(n, 6) + 1))
        rs = [0] + sorted(rng.choice(np.arange(1, m), nr - 1, replace=False).tolist()) + [m] if nr > 1 else [0, m]
        cs = [0] + sorted(rng.choice(np.arange(1, n), nc - 1, replace=False).tolist()) + [n] if nc > 1 else [0, n]
        return GEN(m, n, rs, cs, rng.integers(0, P, (len(rs) - 1) * (len(cs) - 1)).tolist(), P, order)

    A, B = lay(M, N), lay(*((M, N) if op == "N" else (N, M)))
    alpha, beta = [(1.0, 0.0), (2.0, 0.5), (-1.5, 0.0)][(seed // 4) % 3]
    if dtype in ("c128", "c64") and alpha != 1:
        alpha, beta = alpha - 1j, beta and 0.25 + 1j
    return synth.Workload("r", dtype, [synth.Item(A, B, op, alpha, beta)], False, seed=seed), \
        rng.permutation(P).tolist()


def _column_cases():
    """Transposes whose overlay holds rectangles one element wide: blocks one
    longer than the other side's, and a whole matrix of one row."""
    for k, (dtype, op, alpha, beta) in enumerate([("f32", "T", -1.5, 0.25), ("f64", "N", 1.0, 0.0),
                                                  ("c64", "C", 1.0, 0.0), ("c128", "C", 1 - 1j, 0.5)]):
        a, b = ("row", "row") if op != "N" else ("row", "col")
        A = BC(131, 97, 16, 12, 2, 2, "row", a)
        B = BC(*((131, 97) if op == "N" else (97, 131)), 17, 17, 2, 2, "col", b)
        yield synth.Workload(f"columns_{dtype}", dtype, [synth.Item(A, B, op, alpha, beta)], False, seed=60 + k)
    A, B = BC(1, 300, 1, 7, 1, 2, "row", "col"), BC(1, 300, 1, 9, 1, 2, "row", "row")
    yield synth.Workload("one_row", "f32", [synth.Item(A, B, "N", 2.0, 0.0)], False, seed=65)


def _cases():
    for name in synth.WORKLOADS:
        yield synth.workload(name, "small"), None
    for w in short_walk_cases() + stack_cases() + [random_stack_case(s) for s in range(4)]:
        yield w, None
    for s in range(24):
        yield _random_workload(s)
    dtype, op, alpha, beta, A, B, sigma = many_rank_cases()[1]
    yield synth.Workload("many", dtype, [synth.Item(A, B, op, alpha, beta)], False, seed=91), sigma
    for w in _column_cases():
        yield w, None


@pytest.mark.parametrize("k", range(len(list(_cases()))))
def test_direct_rectangles_reproduce_the_oracle(k):
    w, sigma = list(_cases())[k]
    descs, keep = _descs(w)
    x = C.costa_plan_export_direct(w.dtype, descs, sigma)
    assert (x["kind"] == DIRECT).all()
    es, npt, n, P = synth.ITEMSIZE[w.dtype], oracle.NUMPY[w.dtype], len(w.items), w.items[0].A.nranks
    for launch in np.unique(x["launch"]):
        ps = [p for p in x if p["launch"] == launch]
        if int(ps[0]["flags"]) & 1:
            check_tiles(ps, es)
            continue
        assert all(int(p["reserved"]) == 0 for p in ps)
        check_tasks(ps, es)
        assert all((cv == 1).all() for cv in stack_walk_cover(ps, es).values())
    sg = list(range(P)) if sigma is None else sigma
    inv = [sg.index(r) for r in range(P)]
    u = np.uint64 if w.dtype in ("f64", "c128") else np.uint32

    def fills(spec, role, item, labels):
        out, O = [], oracle.OLayout(spec)
        for r in range(P):
            out.append(np.zeros(O.local_elems(labels[r]), dtype=npt))
            oracle.fill(w.dtype, out[-1], w.seed, synth.stream(role, item, r))
        return out

    bufs = [a for i, it in enumerate(w.items) for a in fills(it.A, synth.ROLE_A, i, inv)]
    bufs += [b for i, it in enumerate(w.items) for b in fills(it.B, synth.ROLE_B, i, range(P))]
    hits = [np.zeros(a.size, np.int32) for a in bufs[:n * P]]
    for p in x:
        src, dst = _index(p)
        assert p["dst_buf"] < n * P <= p["src_buf"] < 2 * n * P
        sb, db = bufs[p["src_buf"]], bufs[p["dst_buf"]]
        assert src.min() >= 0 and src.max() < sb.size and dst.min() >= 0 and dst.max() < db.size
        it = w.items[p["item"]]
        alpha, beta = complex(it.alpha), complex(it.beta)
        db[dst] = _combine(w.dtype, sb[src], db[dst] if beta != 0 else None, alpha, beta, it.op == "C")
        hits[p["dst_buf"]][dst] += 1
    for i, it in enumerate(w.items):
        ha = fills(it.A, synth.ROLE_A, i, inv)
        oracle.transform(w.dtype, it.op, it.alpha, it.beta, oracle.OLayout(it.A), ha, oracle.OLayout(it.B),
                         bufs[(n + i) * P:(n + i + 1) * P], sigma)
        want = _written_mask(it, sigma)
        for r in range(P):
            assert np.array_equal(hits[i * P + r], want[r]), "an element of A is not written exactly once"
            assert np.array_equal(bufs[i * P + r].view(u), ha[r].view(u))


@pytest.mark.parametrize("dtype", ["f64", "c128", "f32", "c64"])
def test_both_tile_kernels_are_planned(dtype):
    """Blocks of 12 elements move in tiles of one wave, blocks of 256 in tiles
    of 256 lanes."""
    for block, lanes in ((12, 64), (256, 256)):
        A, B = BC(1024, 768, block, block, 2, 2, "row", "row"), BC(768, 1024, block, block, 2, 2, "col", "row")
        w = synth.Workload("b", dtype, [synth.Item(A, B, "T", 2.0, 0.5)], False, seed=70)
        descs, keep = _descs(w)
        x = C.costa_plan_export_direct(dtype, descs, None)
        assert check_tiles([p for p in x if p["launch"] == 0], synth.ITEMSIZE[dtype]) == lanes


@pytest.mark.parametrize("w", list(_column_cases())[:4], ids=lambda w: w.name)
def test_columns_join_the_launch_of_tiles(w):
    descs, keep = _descs(w)
    x = C.costa_plan_export_direct(w.dtype, descs, None)
    assert (x["nx"] == 1).any() and (x["nx"] > 1).any()
    assert (x["launch"] == 0).all() and (x["flags"] & 1 == 1).all()


# ---------------------------------------------------------------------------
# GPU
# ---------------------------------------------------------------------------
@pytest.mark.gpu
@pytest.mark.parametrize("k", range(len(list(_cases()))))
def test_both_forms_match_the_oracle(k):
    from parity import Case
    w, sigma = list(_cases())[k]
    print(f"both forms: case {k} {w.name} {w.dtype}", flush=True)
    case = Case(w, sigma=sigma)
    for timing in (C.TIMING_AS_CALLED, C.TIMING_MESSAGES):
        case.fill()
        C.costa_timing_enable(timing)
        try:
            case.run()
            t = C.costa_timing_read()
        finally:
            C.costa_timing_enable(False)
        if timing == C.TIMING_AS_CALLED:
            assert t["direct"]["launches"] > 0 and t["pack"]["launches"] == t["unpack"]["launches"] == 0
        case.check_full()


@pytest.mark.gpu
@pytest.mark.parametrize("entry", ["transform", "noalloc"])
def test_overlapping_buffers_take_the_message_form(entry):
    """Two ranks swap the halves of a matrix in place (A's buffers are B's):
    every block is remote, so the message form reads all of B before it
    writes A."""
    M, N = 300, 256
    A = GEN(M, N, [0, M], [0, N // 2, N], [0, 1], 2, "col")
    B = GEN(M, N, [0, M], [0, N // 2, N], [1, 0], 2, "col")
    LA, LB = C.layout_from_spec(A), C.layout_from_spec(B)
    bufs = [torch.rand(M * N // 2, dtype=torch.float64, device="cuda") for _ in range(2)]
    before = [b.clone() for b in bufs]
    print(f"in-place swap: {entry}", flush=True)
    if entry == "transform":
        C.costa_transform("f64", "N", 1.0, 0.0, LA, bufs, LB, bufs)
    else:
        C.costa_transform_batched_noalloc("f64", [dict(op="N", alpha=1.0, beta=0.0, A=LA, A_local=bufs, B=LB,
                                                       B_local=bufs)])
    torch.cuda.synchronize()
    assert torch.equal(bufs[0], before[1]) and torch.equal(bufs[1], before[0])


@pytest.mark.gpu
def test_noalloc_plans_share_the_table_area():
    """Twenty plans of about 1 MB of tables take turns, twice: the later ones
    displace the earlier ones in the 16 MiB table area, and every call finds
    its own."""
    print("noalloc: 20 plans in turn", flush=True)
    calls = []
    for k in range(20):
        A, B = BC(1024, 1000 + k, 24, 8, 2, 2, "row", "col"), BC(1024, 1000 + k, 8, 16, 2, 2, "col", "col")
        LA, LB = C.layout_from_spec(A), C.layout_from_spec(B)
        b = [torch.rand(LB.local_elems(r), dtype=torch.float64, device="cuda") for r in range(4)]
        a = [torch.zeros(LA.local_elems(r), dtype=torch.float64, device="cuda") for r in range(4)]
        want = [torch.zeros_like(t) for t in a]
        C.costa_transform("f64", "N", 1.0, 0.0, LA, want, LB, b)
        calls.append((dict(op="N", alpha=1.0, beta=0.0, A=LA, A_local=a, B=LB, B_local=b), a, want))
    for _ in range(2):
        for d, a, want in calls:
            for t in a:
                t.zero_()
            C.costa_transform_batched_noalloc("f64", [d])
            torch.cuda.synchronize()
            assert all(torch.equal(x, y) for x, y in zip(a, want))


@pytest.mark.gpu
def test_captured_noalloc_call_keeps_its_tables():
    """A captured call replays right after other plans have taken turns in the
    rest of the table area (20 of about 1 MB each)."""
    print("noalloc: captured call, 20 plans between its replays", flush=True)
    LA, LB = C.layout_from_spec(BC(700, 900, 24, 8, 2, 2, "row", "col")), \
        C.layout_from_spec(BC(700, 900, 8, 16, 2, 2, "col", "col"))
    b = [torch.rand(LB.local_elems(r), dtype=torch.float64, device="cuda") for r in range(4)]
    a = [torch.zeros(LA.local_elems(r), dtype=torch.float64, device="cuda") for r in range(4)]
    want = [torch.zeros_like(t) for t in a]
    C.costa_transform("f64", "N", 1.0, 0.0, LA, want, LB, b)
    d = dict(op="N", alpha=1.0, beta=0.0, A=LA, A_local=a, B=LB, B_local=b)
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(stream):
        C.costa_transform_batched_noalloc("f64", [d])
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        C.costa_transform_batched_noalloc("f64", [d])
    for _ in range(2):
        test_noalloc_plans_share_the_table_area()
        for t in a:
            t.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(x, y) for x, y in zip(a, want))


@pytest.mark.gpu
@pytest.mark.parametrize("warm", [False, True])
def test_captured_noalloc_calls_with_device_tables(warm):
    """128 ranks: a call table too large for kernel arguments.  Captured and
    uncaptured calls of one plan with different buffers each move their own."""
    print(f"noalloc: captured calls, 128 ranks, warm={warm}", flush=True)
    A, B = BC(640, 600 + warm, 12, 20, 16, 8, "row", "col"), BC(640, 600 + warm, 16, 12, 8, 16, "col", "row")
    LA, LB = C.layout_from_spec(A), C.layout_from_spec(B)
    calls = []
    for _ in range(3):
        b = [torch.rand(LB.local_elems(r), dtype=torch.float64, device="cuda") for r in range(128)]
        a = [torch.zeros(LA.local_elems(r), dtype=torch.float64, device="cuda") for r in range(128)]
        want = [torch.zeros_like(t) for t in a]
        C.costa_transform("f64", "N", 1.0, 0.0, LA, want, LB, b)
        calls.append((dict(op="N", alpha=1.0, beta=0.0, A=LA, A_local=a, B=LB, B_local=b), a, want))
    small = C.layout_from_spec(BC(40, 40, 8, 8, 2, 2, "row", "col"))
    x = [torch.zeros(small.local_elems(r % 4), dtype=torch.float64, device="cuda") for r in range(8)]
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):  # (the scratch array's address is known before the first capture)
        C.costa_transform_batched_noalloc("f64", [dict(op="N", alpha=1.0, beta=0.0, A=small, A_local=x[:4], B=small,
                                                       B_local=x[4:])])
        if warm:
            C.costa_transform_batched_noalloc("f64", [calls[0][0]])
    torch.cuda.synchronize()
    graphs = []

    def capture(k):
        graphs.append(torch.cuda.CUDAGraph())
        with torch.cuda.graph(graphs[-1], stream=stream):
            C.costa_transform_batched_noalloc("f64", [calls[k][0]])

    def check(k, run):
        d, a, want = calls[k]
        for t in a:
            t.zero_()
        torch.cuda.synchronize()
        run()
        torch.cuda.synchronize()
        assert all(torch.equal(p, q) for p, q in zip(a, want))

    def eager(k):
        check(k, lambda: C.costa_transform_batched_noalloc("f64", [calls[k][0]]))

    capture(0)
    eager(0)
    eager(1)
    check(0, graphs[0].replay)
    capture(1)
    for _ in range(2):
        check(0, graphs[0].replay)
        eager(2)
        check(1, graphs[1].replay)
    eager(0)
