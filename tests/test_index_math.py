"""The kernels' index arithmetic (csrc/index_math.hpp), compiled for the host:
the division by a reciprocal estimate, a lane's way through a tile, the order
of a launch's workgroups."""
import numpy as np
import pytest

pytestmark = pytest.mark.spawns  # builds the stand-in


@pytest.fixture(scope="module")
def standin():
    import standin
    return standin.load()


def _ptr(a):
    return a.ctypes.data


@pytest.mark.parametrize("lanes", [64, 256])
def test_lanes_step_through_every_tile_element(standin, lanes):
    """A lane's steps (one division, then the same additions, and one more
    past a row's end) visit every element of a tile once, at the memory offset
    and LDS slot of its row and column."""
    for rows, length in [(1, 1), (2, 3), (7, 64), (64, 7), (23, 37), (3, 255), (2, 257), (5, 300), (1, 1024), (128, 16)]:
        for ls, lc in ((length | 1, 1), (1, rows | 1)):  # into LDS by rows, out of it by columns
            ld = 2**33 + 3
            seen = np.zeros((rows, length), int)
            for tid in range(lanes):
                steps = -(-rows * length // lanes)
                off, slot = np.empty(steps, np.int64), np.empty(steps, np.int32)
                standin.tile_walk(lanes, tid, length, ld, ls, lc, steps, _ptr(off), _ptr(slot))
                inside = np.arange(steps) * lanes + tid < rows * length
                r, c = off[inside] // ld, off[inside] % ld
                assert (slot[inside] == r * ls + c * lc).all()
                np.add.at(seen, (r, c), 1)
            assert (seen == 1).all()


@pytest.mark.parametrize("ulps", [-1, 0, 1])
def test_division_by_reciprocal_needs_one_step(standin, ulps):
    """The kernels' u / n for u < 2^22 + 1024 (row walks, tiles) and, for
    n >= 2, for u < 2^23 (stacks), with the reciprocal one ulp off either way."""
    rng = np.random.default_rng(5)
    for top, first in (((1 << 22) + 1024, 1), (1 << 23, 2)):
        n = np.concatenate([np.arange(first, 3000), rng.integers(first, top, 3000)]).astype(np.int64)
        for k in (1, 2, 3, 1 << 10, 1 << 20, 1 << 30):
            m = np.minimum(np.minimum(k, (top - 1) // n) * n, top - 1)  # multiples of n, and the last ones
            for u in (m, np.maximum(m - 1, 0), np.minimum(m + 1, top - 1)):
                u32, n32 = u.astype(np.int32), n.astype(np.int32)
                y, x = np.empty_like(u32), np.empty_like(u32)
                standin.divmod(ulps, _ptr(u32), _ptr(n32), _ptr(y), _ptr(x), len(u32))
                assert (y == u // n).all() and (x == u % n).all()


@pytest.mark.parametrize("run", [-1, 0, 4, 16])
def test_workgroup_order_is_a_permutation(standin, run):
    for n in (1, 7, 8, 127, 128, 129, 1000, 4096, 4100):
        out = np.empty(n, np.int32)
        standin.xcd_order(n, run, _ptr(out))
        assert sorted(out.tolist()) == list(range(n))
        if run > 0:  # an XCD (workgroup index modulo 8) takes runs of consecutive tasks
            full = n // (8 * run) * 8 * run
            for x in range(8):
                mine = out[:full][x::8].reshape(-1, run)
                assert (np.diff(mine, axis=1) == 1).all() and (mine[:, 0] % run == 0).all()
