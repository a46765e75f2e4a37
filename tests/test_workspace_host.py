"""Workspace sizes grow with the sizes asked for, also where the launches
change their block sizes: a workspace for the largest case serves the smaller
ones (host only)."""
import ctypes

import pytest

from paper_2501_08174_amd import _lib


def _size(name, *args):
    n = ctypes.c_size_t()
    _lib.call(name, *args, ctypes.byref(n))
    return n.value


def _around(edges):
    return sorted({max(e + d, 0) for e in edges for d in (-8193, -4097, -1025, -257, -2, -1, 0, 1, 2, 257, 1025, 4097, 8193)})


EDGES = [0, 1 << 10, 1 << 12, 1 << 13, 1 << 18, 1 << 20, 1 << 21, 1 << 22, 1 << 24, 1 << 25]


def _non_decreasing(sizes, f):
    got = [f(s) for s in sizes]
    for a, b, x, y in zip(sizes, sizes[1:], got, got[1:]):
        assert x <= y, (a, b, x, y)


@pytest.mark.parametrize("N,V", [(0, 0), (1, 1), (1000, 4), (300000, 16)])
def test_binning_workspace_by_capacity(N, V):
    _non_decreasing(_around(EDGES + [1 << 27, (1 << 32) - 10000]), lambda c: _size("sr_bin_workspace_size", N, V, c))


@pytest.mark.parametrize("cap", [0, 1 << 20, 1 << 26])
def test_binning_workspace_by_pairs(cap):
    _non_decreasing(_around(EDGES), lambda n: _size("sr_bin_workspace_size", n, 1, cap))


def test_tile_order_workspace():
    _non_decreasing(_around(EDGES + [1 << 27]), lambda t: _size("sr_tile_order_workspace_size", t))


def test_compaction_workspace():
    _non_decreasing(_around(EDGES), lambda n: _size("sr_compact_workspace_size", n))
