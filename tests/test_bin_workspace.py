"""The scratch that gs_bin_sort asks for on the CPU: a caller may size it once, for the
largest map and window it will bin, and go on with fewer Gaussians, views or tiles."""
import ctypes
import itertools

import pytest

from tests.test_capi import _views, gs   # noqa: F401 (the fixture)


def _size(gs, n, sizes, cap=65536):
    return gs.lib().gs_bin_sort_workspace_size(n, ctypes.byref(_views(gs, sizes)), cap)


# around the numbers of Gaussians at which the chunks grow, for 1 to 5 views, and beyond
COUNTS = sorted({max(0, e // v + d) for e in (0, 64, 1024, 1 << 14, 1 << 16, 1 << 18, 1 << 20)
                 for v in (1, 2, 3, 5, 40) for d in (-1, 0, 1, 64)} | {500000})


@pytest.mark.parametrize("sizes", [[(16, 16)], [(640, 480)], [(1920, 1080)], [(640, 480), (160, 120)],
                                   [(320, 240)] * 5, [(1280, 960)] * 3, [(160, 120)] * 40,
                                   [(2048, 1024), (2048, 1024), (16, 16)], [(2064, 1024)]])
def test_size_grows_with_the_gaussians(gs, sizes):
    got = [_size(gs, n, sizes) for n in COUNTS]
    assert got[0] > 0
    assert got == sorted(got), [(n, a, b) for n, a, b in zip(COUNTS, got, got[1:]) if b < a]


@pytest.mark.parametrize("n", [1, 1000, 16384, 16385, 20000, 65536, 65537, 200000, (1 << 18) + 1])
def test_size_covers_fewer_and_smaller_views(gs, n):
    full = [(1280, 960), (640, 480), (2048, 1024), (160, 120), (640, 480)]
    top = _size(gs, n, full)
    for k in range(1, len(full) + 1):
        for some in itertools.combinations(full, k):
            assert _size(gs, n, list(some)) <= top, some
    assert _size(gs, n, [(640, 480)] * 5) <= top
    many = [_size(gs, n, [(640, 480)] * k) for k in range(1, 65)]
    assert many == sorted(many)
    tall = [_size(gs, n, [(1024, 16 * k)]) for k in (1, 7, 100, 127, 128, 129, 300)]   # past 8,192 tiles
    assert tall[0] > 0 and tall == sorted(tall)


def test_size_grows_with_the_capacity(gs):
    got = [_size(gs, 20000, [(640, 480)], cap) for cap in (0, 1, 1000, 65536, 1 << 24)]
    assert got == sorted(got)
