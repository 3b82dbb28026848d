"""The tile kernels' own choice of pixels per lane (from the number of tiles)
renders what every set value renders: images, final transmittances, last
splats and losses bit for bit, gradients up to the order of their atomic additions
(needs an MI355X)."""
import numpy as np
import pytest
import torch

from paper_2409_09295_amd import scenes
from tests.gpu_helpers import assert_same_up_to_order, np_

pytestmark = pytest.mark.gpu

DEV = "cuda"


def _views_of(gs, tiles):
    """Views of `tiles` tiles in all: a strip of 100 tile columns and a rest."""
    rows, rest = divmod(tiles, 100)
    sizes = ([(1600, 16 * rows)] if rows else []) + ([(16 * rest, 16)] if rest else [])
    views = gs.Views([scenes.pinhole(w, h, 0.8 * w) for w, h in sizes])
    assert views.n_tiles == tiles
    return views


def _step(gs, g, views, target, ppl):
    gs.gs_set_tuning(gs.GS_TUNE_FWD_PIXELS_PER_LANE, ppl)
    gs.gs_set_tuning(gs.GS_TUNE_BWD_PIXELS_PER_LANE, ppl)
    try:
        from paper_2409_09295_amd.rasterizer import Rasterizer
        r = Rasterizer(g.n, views)
        dl = torch.empty(3 * views.n_pixels, device=DEV)
        loss = torch.zeros(1, dtype=torch.float64, device=DEV)
        grads = gs.Grads.zeros_like(g, views.n_views)
        r.forward_l1(g, target, dl, loss)
        r.backward(g, dl, grads)
        torch.cuda.synchronize()
        return r, dl, loss, grads
    finally:
        gs.gs_set_tuning(gs.GS_TUNE_FWD_PIXELS_PER_LANE, 0)
        gs.gs_set_tuning(gs.GS_TUNE_BWD_PIXELS_PER_LANE, 0)


@pytest.mark.parametrize("tiles", [1, 1999, 2000, 2399, 2400, 4999, 5000, 7999, 8000])
def test_chosen_pixels_per_lane_match_every_set_value(gs, tiles):
    print(f"tiles {tiles}", flush=True)
    views = _views_of(gs, tiles)
    g = gs.Gaussians.from_map(scenes.random_cloud(3000, 1, seed=tiles))
    gen = torch.Generator(device=DEV).manual_seed(tiles)
    target = torch.rand(3 * views.n_pixels, generator=gen, device=DEV)
    r0, dl0, loss0, g0 = _step(gs, g, views, target, 0)
    for ppl in (1, 2, 4):
        r, dl, loss, gr = _step(gs, g, views, target, ppl)
        for a, b in ((r.image, r0.image), (r.final_T, r0.final_T), (r.n_contrib, r0.n_contrib), (dl, dl0)):
            torch.testing.assert_close(a, b, rtol=0, atol=0)
        assert loss.item() == loss0.item()
        for name in ("means", "log_scales", "quats", "opacity_logits", "sh", "xi"):
            assert_same_up_to_order(name, np_(getattr(gr, name)), np_(getattr(g0, name)))


def test_reported_default(gs):
    assert gs.gs_get_tuning(gs.GS_TUNE_FWD_PIXELS_PER_LANE) == 1
    assert gs.gs_get_tuning(gs.GS_TUNE_BWD_PIXELS_PER_LANE) == 1
