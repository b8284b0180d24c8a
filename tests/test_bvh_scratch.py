"""Sizes of the tree build's scratch arrays, for the counts that its kernels
are launched with (on the CPU: the library's own size functions)."""

import ctypes

import pytest

from paper_2210_06158_amd import dof


def _fn(name, restype):
    f = getattr(dof.lib(), name)
    f.restype, f.argtypes = restype, [ctypes.c_int64]
    return f


def _counts():
    near = [1, 1024, 2048, 4096, 65536, 128 * 1024, 256 * 1024, 512 * 1024, 1024 * 1024, 1 << 24, (1 << 31) - 2]
    return sorted({n + d for n in near for d in (-1, 0, 1) if n + d >= 1} | {3 ** k * 1000 + 7 for k in range(13)})


def test_the_sorts_words_hold_every_tile():
    """hist: the key blocks' rows of 8 x 256 counts (a row per 1024 references,
    at most 256) and one of places, 64 tickets, and 8 x 256 look-back words per
    tile; its size never shrinks as a scene grows."""
    tile, words = _fn("_ZN3dof9sort_tileEl", ctypes.c_int), _fn("_ZN3dof10sort_wordsEl", ctypes.c_int64)
    last = 0
    for n in _counts():
        rows = min(256, -(-n // 1024))
        assert words(n) >= (rows + 1) * 2048 + 64 + 2048 * -(-n // tile(n)), n
        assert words(n) >= last, n
        last = words(n)


def test_the_trees_exits_fit_the_buffers_that_they_reuse():
    """keys_tmp and ids_tmp after the sort: 256 records of 32 bytes per block of
    1024 leaves; up to 64 blocks two rounds of at most 194 records per 1024
    entries behind them, beyond that the merged blocks' records in ids_tmp
    (4 bytes a reference) and two rounds of those in the first.  hist: both
    levels' counts and offsets."""
    words, bytes_ = _fn("_ZN3dof10sort_wordsEl", ctypes.c_int64), _fn("_ZN3dof14keys_tmp_bytesEl", ctypes.c_int64)
    for n in _counts():
        blocks = -(-n // 1024)
        assert bytes_(n) >= 8 * n and bytes_(n) % 16 == 0
        if blocks <= 64:
            top = -(-blocks * 194 // 1024) * 194
            assert bytes_(n) >= 32 * (256 * blocks + 2 * top), n
            assert words(n) >= 2 * blocks + 1
        else:
            merges = -(-blocks * 194 // 1024)
            assert 4 * n >= 32 * 256 * merges, n
            first = -(-merges * 194 // 1024) * 194    # records of the first round
            second = -(-first // 1024) * 194
            pong = 256 * -(-merges // 2)
            assert first <= pong and 32 * (pong + second) <= bytes_(n), n
            assert words(n) >= 2 * blocks + 1 + 2 * merges + 1, n
