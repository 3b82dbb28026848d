"""The reverse walk of launches of few tiles (every list in quarters, one quadrant per
workgroup) against one wavefront per quadrant, at list lengths around its quarters and
batches and at the limit of tiles, within the parity contract of gradients (needs an
MI355X)."""
import math

import pytest
import torch

from paper_2409_09295_amd import scenes
from tests.gpu_helpers import assert_grad_close, np_

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _grads(gs, g, views, ppl, bg):
    from paper_2409_09295_amd.rasterizer import Rasterizer
    gs.gs_set_tuning(gs.GS_TUNE_BWD_PIXELS_PER_LANE, ppl)
    try:
        r = Rasterizer(g.n, views)
        r.forward(g, bg)
        gen = torch.Generator(device=DEV).manual_seed(g.n)
        dl = torch.randn(3 * views.n_pixels, generator=gen, device=DEV) / views.n_pixels
        grads = gs.Grads.zeros_like(g, views.n_views)
        r.backward(g, dl, grads, 0, bg)
        torch.cuda.synchronize()
        return grads, r
    finally:
        gs.gs_set_tuning(gs.GS_TUNE_BWD_PIXELS_PER_LANE, 0)


@pytest.mark.parametrize("n,sizes,faint", [
    (1, [(16, 16)], False), (3, [(16, 16)], True), (4, [(17, 9)], True), (5, [(16, 16)], True),
    (127, [(16, 16)], True), (512, [(16, 16)], True), (513, [(16, 16)], True),
    (1030, [(30, 20)], True), (3000, [(16, 16)], True), (3000, [(40, 24), (16, 16), (9, 70)], False),
    (3000, [(1600, 160)], False), (3000, [(1600, 160), (16, 16)], False)])   # 1,000 and 1,001 tiles
def test_quarters_match_whole_lists(gs, n, sizes, faint):
    print(f"n {n} {sizes}", flush=True)
    views = gs.Views([scenes.pinhole(w, h, 0.8 * w) for w, h in sizes])
    g = gs.Gaussians.from_map(scenes.random_cloud(n, 1, seed=n))
    if faint:   # no pixel ends early: the lists are walked whole
        g.opacity_logits -= 5.0
    bg = (0.3, 0.1, 0.7)
    ref, r = _grads(gs, g, views, 1, bg)
    got, _ = _grads(gs, g, views, 0, bg)
    print("  longest walk", int(r.n_contrib.max()), flush=True)
    for name in ("means", "log_scales", "quats", "opacity_logits", "sh", "xi"):
        assert_grad_close(name, np_(getattr(got, name)), np_(getattr(ref, name)))


@pytest.mark.parametrize("size,n,at", [((16, 16), 40, 25), ((40, 24), 400, 250), ((16, 16), 40, 39)])
def test_infinite_colour_that_no_pixel_blends(gs, size, n, at):
    """A splat of infinite colour between four pixel centres, at 2 / 255 in its middle and
    below 1 / 255 at each centre: it reaches a quadrant and no pixel of it blends it, so
    image and gradients are finite, as they are without the quarters."""
    w, h = size
    f = 0.8 * w
    g = gs.Gaussians.from_map(scenes.random_cloud(n, 0, seed=n, box=((-1, 1), (-1, 1), (2, 4))))
    g.opacity_logits -= 4.0   # lists are walked to the end
    depth = g.means[2].sort().values
    g.means[2] = depth        # list position = index, wherever a list holds all
    z = float(depth[at])
    g.means[0, at], g.means[1, at] = z * (4.0 - w / 2) / f, z * (4.0 - h / 2) / f
    g.log_scales[:, at] = -12.0   # the 0.3 pixels^2 of the filter alone
    o = 2.0 / 255.0
    g.opacity_logits[at] = math.log(o / (1.0 - o))
    g.sh[:, 0, at] = math.inf
    views = gs.Views([scenes.pinhole(w, h, f)])
    ref, r = _grads(gs, g, views, 1, (0.2, 0.5, 0.1))
    got, r = _grads(gs, g, views, 0, (0.2, 0.5, 0.1))
    assert bool(torch.isinf(r.proj.rgb_depth[0, at, :3]).all()) and int(r.proj.radius[0, at]) > 0
    assert bool(torch.isfinite(r.image).all())
    for name in ("means", "log_scales", "quats", "opacity_logits", "sh", "xi"):
        a, b = np_(getattr(got, name)), np_(getattr(ref, name))
        assert (abs(b) < math.inf).all() and (abs(a) < math.inf).all(), name
        assert_grad_close(name, a, b)


@pytest.mark.parametrize("sizes", [[(40, 24), (16, 16), (9, 70)], [(1600, 160)]])
def test_quarters_in_tile_id_order(gs, sizes):
    views = gs.Views([scenes.pinhole(w, h, 0.8 * w) for w, h in sizes])
    g = gs.Gaussians.from_map(scenes.random_cloud(3000, 1, seed=5))
    bg = (0.3, 0.1, 0.7)
    ref, _ = _grads(gs, g, views, 1, bg)
    gs.gs_set_tuning(gs.GS_TUNE_BWD_SCHEDULE, gs.GS_SCHEDULE_TILE_ID)
    try:
        got, _ = _grads(gs, g, views, 0, bg)
    finally:
        gs.gs_set_tuning(gs.GS_TUNE_BWD_SCHEDULE, 0)
    for name in ("means", "log_scales", "quats", "opacity_logits", "sh", "xi"):
        assert_grad_close(name, np_(getattr(got, name)), np_(getattr(ref, name)))
