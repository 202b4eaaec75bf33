"""What the host schedules for the GPU, checked without one."""
import ctypes as C

import numpy as np
import pytest

from paper_2601_04904_amd import _lib


def tile_order(tiles, k):
    """(product, tile) pairs of a launch's order, padding left out."""
    tiles, k = np.ascontiguousarray(tiles, np.int32), np.ascontiguousarray(k, np.int32)
    i32, u64 = C.POINTER(C.c_int32), C.POINTER(C.c_uint64)
    args = (len(tiles), tiles.ctypes.data_as(i32), k.ctypes.data_as(i32))
    n = _lib.lib().bt_si_sq_diag_tile_order(*args, None, 0)
    out = np.empty(n, np.uint64)
    assert _lib.lib().bt_si_sq_diag_tile_order(*args, out.ctypes.data_as(u64), n) == n
    out = out[out != np.uint64(2 ** 64 - 1)]
    return (out >> np.uint64(32)).astype(np.int64), (out & np.uint64(2 ** 32 - 1)).astype(np.int64)


@pytest.mark.parametrize("count,last", [(1, 1), (7, 2049), (130, 5), (2 ** 21 + 3, 1)])
def test_every_tile_of_a_launch_once(count, last):
    """Every tile of every product exactly once: products past 2^21 in one launch, and a
    product of more than 2^11 tiles."""
    tiles = np.ones(count, np.int64)
    tiles[-1] = last
    p, t = tile_order(tiles, 8 + 100 * (np.arange(count) % 3))
    assert len(p) == tiles.sum()
    at = np.lexsort((t, p))
    first = np.concatenate([[0], np.cumsum(tiles)[:-1]])
    assert np.array_equal(p[at], np.repeat(np.arange(count), tiles))
    assert np.array_equal(t[at], np.arange(len(p)) - first[p[at]])


@pytest.mark.parametrize("specs", [[dict(n=64, b=512, a=0, partitions=8)], [dict(n=16, b=32, a=0, partitions=4)],
                                   [dict(n=9, b=100, a=37, partitions=2), dict(n=7, b=300, a=300)] * 3])
def test_handle_size_does_not_depend_on_the_tuning_table(specs):
    """Memory sized under one table holds a handle created under another."""
    from paper_2601_04904_amd import solver as S
    saved = S.tune_table()
    try:
        sizes = []
        for v in range(-1, _lib.BT_TILE_SHAPES):
            S.set_tune_table([v] * _lib.BT_TUNE_ENTRIES)
            sizes.append(S.batch_workspace_bytes(specs))
        assert len(set(sizes)) == 1, sizes
    finally:
        S.set_tune_table(saved)


@pytest.mark.parametrize("m,n,k,count", [(32, 32, 32, 1), (128, 128, 128, 3), (100, 37, 100, 2), (512, 512, 512, 32)])
@pytest.mark.parametrize("mixed", [0, 1])
def test_a_table_entry_is_taken(m, n, k, count, mixed):
    """Every launch takes the shape that its class has in the table, small launches too;
    without an entry small launches take the 16 x 16 tiles."""
    from paper_2601_04904_amd import solver as S
    shape = _lib.lib().bt_si_sq_diag_launch_shape
    saved = S.tune_table()
    try:
        for v in range(_lib.BT_TILE_SHAPES):
            S.set_tune_table([v] * _lib.BT_TUNE_ENTRIES)
            assert shape(m, n, k, count, mixed) == v
        S.set_tune_table([-1] * _lib.BT_TUNE_ENTRIES)
        assert (shape(m, n, k, count, mixed) == _lib.BT_TILE_SHAPES) == (count < 32)
    finally:
        S.set_tune_table(saved)


def panels(d):
    """Launches of blocks of d alone: a panel of 16 columns each, and one to write the result."""
    return 1 if d <= 112 else -(-d // 16) + 1


@pytest.mark.parametrize("sizes,together", [
    ([(256, 1), (512, 1)], True), ([(256, 16), (512, 1)], True), ([(256, 64), (512, 1)], False),
    ([(256, 64), (1024, 1)], False), ([(128, 32), (600, 1)], True), ([(128, 64), (600, 1)], False),
    ([(512, 32), (600, 1)], True), ([(512, 64), (600, 1)], False), ([(128, 256), (256, 1)], True),
    ([(120, 1), (200, 1), (300, 1)], True)])
def test_panel_launches_are_shared_by_few_blocks_only(sizes, together):
    d = np.repeat([s for s, _ in sizes], [c for _, c in sizes]).astype(np.int32)
    got = _lib.lib().bt_si_sq_diag_inverse_launches(len(d), d.ctypes.data_as(C.POINTER(C.c_int32)))
    assert got == (panels(max(d)) if together else sum(panels(s) for s, _ in sizes))


def test_panel_launches_next_to_small_blocks_and_of_three_shapes():
    def count(sizes):
        d = np.repeat([s for s, _ in sizes], [c for _, c in sizes]).astype(np.int32)
        return _lib.lib().bt_si_sq_diag_inverse_launches(len(d), d.ctypes.data_as(C.POINTER(C.c_int32)))
    assert count([(40, 3), (100, 2), (257, 1)]) == 2 + panels(257)
    # the blocks of 128 go with those of 256 where these stay apart from the largest
    assert count([(128, 200), (256, 100), (1024, 1)]) == panels(256) + panels(1024)
    assert count([(128, 200), (256, 1), (1024, 1)]) == panels(128) + panels(1024)
