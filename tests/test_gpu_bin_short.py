"""gs_bin_sort's short path (few entries, few tiles) at the edges of its range
against the general path: the same splats followed by culled ones that push the
call over the limit bin to the same lists, ranges, tile order and key count
(needs an MI355X)."""
import numpy as np
import pytest
import torch

from paper_2409_09295_amd import scenes
from tests.gpu_helpers import u32

pytestmark = pytest.mark.gpu
DEV = "cuda"
LIMIT = 1 << 18   # Gaussians of the short path (and 1 << 20 entries, 16,384 tiles)


def _splats(n, cam, seed, pad=0):
    sp = scenes.random_splats(n, [cam], seed, sigma_px=(0.6, 8.0), cull_frac=0.3, depth_ties=0.05)
    if pad:
        z = lambda a: np.concatenate([a, np.zeros((1, pad) + a.shape[2:], a.dtype)], 1)
        sp = scenes.SplatSet(z(sp.xy), z(sp.conic_opacity), z(sp.rgb_depth), z(sp.radius), sp.cams)
    return sp


def _bin(gs, sp, cam, capacity, sync=True, order=True):
    views = gs.Views([cam])
    proj = gs.Projected.from_splats(sp)
    n = sp.radius.shape[1]
    bins = gs.Bins.empty(capacity, views.n_tiles, order=order)
    bins.queue.fill_(7)
    for t in (bins.values, bins.ranges, bins.keys):
        t.fill_(-1)
    ws = gs.workspace(gs.gs_bin_sort_workspace_size(n, views, capacity))
    try:
        count = gs.gs_bin_sort(proj, n, views, bins, ws, sync=sync)
    except gs.GsError as e:
        assert e.status == gs.GS_ERR_CAPACITY
        count = -e.required
    torch.cuda.synchronize()
    assert int(bins.queue.abs().sum()) == 0
    return bins, count, int(u32(bins.n_keys)[0])


@pytest.mark.parametrize("n,W,H", [(1, 16, 16), (63, 40, 20), (64, 160, 120), (16384, 160, 120),
                                   (16385, 320, 240), (65536, 320, 240), (65537, 100, 70),
                                   (LIMIT, 640, 480), (20000, 2048, 1024), (3000, 16, 16), (3000, 64, 32)])
def test_short_path_matches_the_general_path(gs, n, W, H):
    print(f"n {n} {W}x{H}", flush=True)
    cam = scenes.pinhole(W, H, 0.8 * W)
    few = _splats(n, cam, seed=n)
    many = _splats(n, cam, seed=n, pad=LIMIT + 1 - n)
    _, need, _ = _bin(gs, many, cam, 1)
    need = abs(need)
    a, ca, ka = _bin(gs, few, cam, need + 1)
    b, cb, kb = _bin(gs, many, cam, need + 1)
    assert ca == cb == ka == kb == need
    for x, y in ((a.values, b.values), (a.keys, b.keys), (a.ranges, b.ranges), (a.order, b.order)):
        assert torch.equal(x, y)
    c, _, kc = _bin(gs, few, cam, need + 1, sync=False, order=False)
    assert kc == need and torch.equal(c.values, a.values) and torch.equal(c.ranges, a.ranges)
    if need > 1:   # one slot short: nothing emitted, the identity order, the count reported
        for sync in (True, False):
            d, cd, kd = _bin(gs, few, cam, need - 1, sync=sync)
            assert kd == need and (not sync or cd == -need)
            assert int(d.ranges.abs().sum()) == 0 and int((d.values + 1).abs().sum()) == 0
            assert torch.equal(d.order, torch.arange(d.order.numel(), dtype=torch.int32, device=DEV))


@pytest.mark.parametrize("n,sizes", [(5000, [(100, 70), (320, 240), (16, 16)]),
                                     (4000, [(2048, 1024), (2048, 1024)]),              # 16,384 tiles
                                     (4000, [(2048, 1024), (2048, 1024), (16, 16)]),    # past them
                                     (LIMIT, [(160, 120)] * 4), (LIMIT, [(160, 120)] * 5)])
def test_short_path_views_of_several_sizes(gs, n, sizes):
    """Several views share the matrix: each view binned alone gives its part."""
    print(f"n {n} {sizes}", flush=True)
    cams = [scenes.pinhole(w, h, 0.8 * w) for w, h in sizes]
    sp = scenes.random_splats(n, cams, seed=4, sigma_px=(0.6, 4.0))
    views = gs.Views(cams)
    cap = 1 << 24
    bins = gs.Bins.empty(cap, views.n_tiles)
    ws = gs.workspace(gs.gs_bin_sort_workspace_size(n, views, cap))
    gs.gs_bin_sort(gs.Projected.from_splats(sp), n, views, bins, ws)
    first = 0
    for v, cam in enumerate(cams):
        one = scenes.SplatSet(*[a[v:v + 1] for a in (sp.xy, sp.conic_opacity, sp.rgb_depth, sp.radius)], [cam])
        alone, _, k = _bin(gs, one, cam, cap)
        tiles = alone.ranges.shape[0]
        r = bins.ranges[first:first + tiles].long()
        own = alone.ranges.long()
        assert torch.equal(r[:, 1] - r[:, 0], own[:, 1] - own[:, 0])
        s = int(r[r[:, 1] > r[:, 0]].min())
        assert torch.equal(bins.values[s:s + k] - v * n, alone.values[:k])
        first += tiles


@pytest.mark.parametrize("n", [255, 256, 257, 512, 513, 1024, 1025, 2048, 2049, 4096, 4097])
def test_short_path_list_lengths(gs, n):
    """One tile, every list length at which another sort takes over."""
    print(f"n {n}", flush=True)
    cam = scenes.pinhole(16, 16, 12.0)
    sp = scenes.random_splats(n, [cam], seed=n, sigma_px=(0.6, 8.0), cull_frac=0.0, depth_ties=0.1)
    sp.xy[...] = np.clip(sp.xy, 1.0, 15.0)
    pad = LIMIT + 1 - n
    z = lambda a: np.concatenate([a, np.zeros((1, pad) + a.shape[2:], a.dtype)], 1)
    many = scenes.SplatSet(z(sp.xy), z(sp.conic_opacity), z(sp.rgb_depth), z(sp.radius), sp.cams)
    a, ca, _ = _bin(gs, sp, cam, n)
    b, cb, _ = _bin(gs, many, cam, n)
    assert ca == cb == n
    assert torch.equal(a.values, b.values) and torch.equal(a.keys, b.keys)
