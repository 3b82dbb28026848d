"""The depth kernels at the edges of their tiles: belief propagation's
two-iteration tiles (8x4 pixels) with remainders, odd and even iteration counts,
and the cost volume's workgroups of 16 pixels (needs an MI355X)."""
import numpy as np
import pytest
import torch

from paper_2409_09295_amd import scenes
from tests.gpu_helpers import np_
from tests.test_gpu_bp import _compare, _gpu_bp

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("iters", [1, 2, 3])
@pytest.mark.parametrize("h,w", [(1, 1), (4, 8), (5, 9), (3, 25), (12, 7), (1, 33)])
def test_bp_tile_edges(gs, h, w, iters):
    rng = np.random.default_rng(1000 * iters + 40 * h + w)
    cost = (rng.random((64, h, w)) * 0.3).astype(np.float32)
    cost[rng.random((64, h, w)) < 0.02] = np.inf
    labels, depth = _gpu_bp(gs, cost, 0.01, 0.08, iters)
    _compare(labels, cost, 0.01, 0.08, iters)
    np.testing.assert_array_equal(depth, (0.25 + 24.75 * labels.astype(np.float32) / 63).astype(np.float32))


def test_bp_workspace_needs_only_float_alignment(gs):
    h, w = 9, 11
    rng = np.random.default_rng(2)
    cost = (rng.random((64, h, w)) * 0.3).astype(np.float32)
    ref, _ = _gpu_bp(gs, cost, 0.01, 0.08, 4)
    c = torch.from_numpy(cost).to(DEV)
    ws = gs.workspace(gs.gs_bp_workspace_size(h, w) + 16)[4:]
    labels = torch.full((h, w), -1, dtype=torch.int32, device=DEV)
    gs.gs_bp_labels(c, h, w, 0.01, 0.08, 4, 1.0, labels, None, ws)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(np_(labels), ref)


@pytest.mark.parametrize("k,H,W", [(2, 4, 4), (3, 12, 20), (2, 20, 68), (4, 16, 64)])
def test_cost_volume_winner_is_the_first_minimum(gs, k, H, W):
    cams = [scenes.pinhole(W, H, 0.8 * W, t=np.array([0.05 * i, 0.02 * i, 0.0])) for i in range(k)]
    views = gs.Views(cams)
    gen = torch.Generator(device=DEV).manual_seed(k * W)
    rgb = torch.rand(k, 3, H, W, generator=gen, device=DEV)
    cost = torch.empty(64, H // 4, W // 4, device=DEV)
    depth = torch.empty(H // 4, W // 4, device=DEV)
    ws = gs.workspace(gs.gs_cost_volume_workspace_size(k, H, W))
    gs.gs_cost_volume_wta(rgb, views, cost, depth, ws)
    only = torch.empty_like(depth)
    gs.gs_cost_volume_wta(rgb, views, None, only, ws)
    torch.cuda.synchronize()
    c = np_(cost)
    first = c.argmin(0)
    want = np.where(np.isfinite(c).any(0), (0.25 + 24.75 * first.astype(np.float32) / 63).astype(np.float32), 0.0)
    np.testing.assert_array_equal(np_(depth), want.astype(np.float32))
    np.testing.assert_array_equal(np_(only), np_(depth))
