"""The volume matrix of two block-cyclic layouts at the ends of what its
kernel's integers hold, on the CPU: the library's host code and the kernel's
own count of overlaps over the stand-in of the HIP runtime, against a plain
count."""
import numpy as np
import pytest

pytestmark = pytest.mark.spawns  # builds the stand-in


@pytest.fixture(scope="module")
def standin():
    import standin
    return standin.load()


def _want(n, a, b):
    """Elements by (process of b, process of a); a and b are (block, processes)."""
    h = np.zeros((b[1], a[1]), np.int64)
    for i in range(n):
        h[i // b[0] % b[1], i // a[0] % a[1]] += 1
    return h


@pytest.mark.parametrize("big", [97, 2**30, 2**31 - 1, 2**31, 2**32, 2**33 - 1, 2**61, 2**62 - 1, 2**62, 2**62 + 2**32,
                                 2**63 - 1])
@pytest.mark.parametrize("side", ["source", "target", "both"])
def test_blocks_longer_than_the_matrix(standin, big, side):
    S, C = standin, standin.C
    m, n = 97, 60
    a = (big, 3) if side != "source" else (8, 3)
    b = (big, 3) if side != "target" else (5, 3)
    A = C.Layout.block_cyclic(m, n, a[0], 7, 3, 2, "row", "col")
    B = C.Layout.block_cyclic(m, n, b[0], 9, 3, 2, "row", "col")
    hr, hc = _want(m, a, b), _want(n, (7, 2), (9, 2))
    want = np.einsum("ij,kl->ikjl", hr, hc).reshape(6, 6)
    V = C.costa_volume_matrix(A, B, "N", stream=S.stream())
    S.check()
    assert np.array_equal(V, want)


@pytest.mark.parametrize("n", [5, 65536, 65537, 2**31 - 65536, 2**31 - 65535, 2**31 - 2])
def test_a_lane_ends_at_the_last_block(standin, n):
    """64 workgroups of 1024 lanes step through up to 2^31 - 2 blocks."""
    step = 65536
    for first in (0, 1, step - 1):
        assert standin.lane_volume(n, first, step) == max(0, -(-(n - first) // step))
