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
from test_plan_replay import DIRECT, _descs, _written_mask, check_tasks, stack_walk_cover

C = pytest.importorskip("paper_2106_06601_amd")
BC, GEN, SL = synth.BlockCyclic, synth.General, synth.ScaLapack


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


def _cases():
    for name in synth.WORKLOADS:
        yield synth.workload(name, "small"), None
    for w in short_walk_cases() + stack_cases() + [random_stack_case(s) for s in range(4)]:
        yield w, None
    for s in range(24):
        yield _random_workload(s)
    dtype, op, alpha, beta, A, B, sigma = many_rank_cases()[1]
    yield synth.Workload("many", dtype, [synth.Item(A, B, op, alpha, beta)], False, seed=91), sigma


@pytest.mark.parametrize("k", range(len(list(_cases()))))
def test_direct_rectangles_reproduce_the_oracle(k):
    w, sigma = list(_cases())[k]
    descs, keep = _descs(w)
    x = C.costa_plan_export_direct(w.dtype, descs, sigma)
    assert (x["kind"] == DIRECT).all()
    es, npt, n, P = synth.ITEMSIZE[w.dtype], oracle.NUMPY[w.dtype], len(w.items), w.items[0].A.nranks
    check_tasks(x, es)
    for launch in np.unique(x["launch"]):
        ps = [p for p in x if p["launch"] == launch]
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
