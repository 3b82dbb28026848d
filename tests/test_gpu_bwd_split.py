"""The reverse walk of launches of few tiles (every list in quarters, one quadrant per
workgroup) against one wavefront per quadrant, at list lengths around its quarters and
batches and at the limit of tiles, within the parity contract of gradients (needs an
MI355X)."""
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
