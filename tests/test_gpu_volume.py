"""The one-launch volume kernel of two block-cyclic layouts against a plain
count, where it can go wrong: windows that start inside blocks, either side the
finer one, equal blocks, several workgroups, one process, rank maps that leave
ranks out, the largest rank count and histogram it takes and the first past
them (the two-launch kernels), and calls that alternate with the overlay
kernel on the same scratch memory."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2106_06601_amd as C

SL, GEN = synth.ScaLapack, synth.General

# (rows, cols, op, [A: mb nb prow pcol rsrc csrc i0 j0], [B: the same])
CASES = {
    "one_process": (50, 70, "N", [7, 9, 1, 1, 0, 0, 0, 0], [5, 5, 1, 1, 0, 0, 3, 2]),
    "windows": (999, 1001, "N", [32, 24, 3, 2, 1, 1, 17, 50], [20, 64, 2, 3, 1, 2, 63, 5]),
    "transposed": (640, 900, "T", [40, 100, 4, 2, 2, 0, 0, 99], [8, 12, 2, 4, 0, 3, 11, 0]),
    "source_coarser": (4000, 300, "C", [3, 2, 5, 2, 0, 0, 1, 1], [100, 700, 2, 5, 1, 4, 250, 0]),
    "equal_blocks": (512, 512, "N", [16, 16, 4, 4, 0, 0, 0, 0], [16, 16, 4, 4, 0, 0, 8, 8]),
    "many_blocks": (20000, 9001, "N", [1, 2, 4, 4, 0, 0, 0, 0], [3, 1, 4, 4, 0, 0, 2, 1]),
    "ranks_256": (3000, 2000, "N", [10, 10, 16, 16, 5, 7, 0, 0], [7, 30, 8, 32, 1, 2, 4, 4]),
    "ranks_272": (1500, 1500, "N", [10, 10, 16, 17, 5, 7, 0, 0], [7, 30, 17, 16, 1, 2, 4, 4]),
    "histogram_4097": (3000, 60, "N", [1, 10, 64, 1, 0, 0, 0, 0], [2, 5, 64, 1, 3, 0, 1, 1]),
}


def _count(n, a, b):
    """Elements by (process of b, process of a) of one dimension; a and b are
    (block, processes, source process, offset)."""
    i = np.arange(n)
    own = lambda s: ((i + s[3]) // s[0] + s[2]) % s[1]  # noqa: E731
    h = np.zeros((b[1], a[1]), np.int64)
    np.add.at(h, (own(b), own(a)), 1)
    return h


@pytest.mark.parametrize("mapped", [False, True])
@pytest.mark.parametrize("name", list(CASES))
def test_volume_of_dealt_layouts(name, mapped):
    m, n, op, a, b = CASES[name]
    print(f"volume {name} mapped={mapped}", flush=True)
    P = a[2] * a[3]
    world = P + 3 if mapped else P
    rng = np.random.default_rng(11)
    maps = [rng.permutation(world)[:P].tolist() if mapped else None for _ in range(2)]

    def window(s, rows, cols, rank_map):
        M, N = rows + s[6], cols + s[7]
        lld = max(1, -(-(-(-M // s[0])) // s[2]) * s[0])
        full = C.layout_from_spec(SL(M, N, s[0], s[1], s[4], s[5], lld, s[2], s[3], "row",
                                     world=world if mapped else 0, rank_map=rank_map))
        return full.submatrix(s[6], s[7], rows, cols)

    tr = op != "N"
    A, B = window(a, m, n, maps[0]), window(b, *((n, m) if tr else (m, n)), maps[1])
    bd = [(b[0], b[2], b[4], b[6]), (b[1], b[3], b[5], b[7])]
    hr = _count(m, (a[0], a[2], a[4], a[6]), bd[1] if tr else bd[0])
    hc = _count(n, (a[1], a[3], a[5], a[7]), bd[0] if tr else bd[1])
    want = np.zeros((world, world), np.int64)
    for s in range(P):
        br, bc = (s % b[2], s // b[2]) if mapped else (s // b[3], s % b[3])
        for t in range(P):
            ar, ac = (t % a[2], t // a[2]) if mapped else (t // a[3], t % a[3])
            r, c = (bc, br) if tr else (br, bc)
            want[maps[1][s] if mapped else s, maps[0][t] if mapped else t] = hr[r, ar] * hc[c, ac]
    G = C.layout_from_spec(GEN(5, 4, [0, 2, 5], [0, 1, 4], [0, 1, 1, 0], 2, "col"))
    for _ in range(2):
        assert np.array_equal(C.costa_volume_matrix(A, B, op), want)
    assert C.costa_volume_matrix(G, G, "N").tolist() == [[11, 0], [0, 9]]  # the overlay kernel in between
    assert np.array_equal(C.costa_volume_matrix(A, B, op), want)


@pytest.mark.parametrize("big", [2**31 - 1, 2**33 - 1, 2**62, 2**63 - 1])
def test_volume_of_blocks_longer_than_the_matrix(big):
    """(block size 2^62: its low 32 bits are zero)"""
    print(f"volume, blocks of {big}", flush=True)
    m, n = 97, 60
    for a, b in ((big, 5), (8, big), (big, big)):
        A = C.Layout.block_cyclic(m, n, a, 7, 3, 2, "row", "col")
        B = C.Layout.block_cyclic(m, n, b, 9, 3, 2, "row", "col")
        hr, hc = _count(m, (a, 3, 0, 0), (b, 3, 0, 0)), _count(n, (7, 2, 0, 0), (9, 2, 0, 0))
        want = np.einsum("ij,kl->ikjl", hr, hc).reshape(6, 6)
        assert np.array_equal(C.costa_volume_matrix(A, B, "N"), want)
