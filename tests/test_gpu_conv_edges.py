"""The U-Net's convolution kernels at the edges of their tiles, strips and
channel groups against the FP64 oracle (needs an MI355X).  Tolerance: FP32
accumulation error within 1e-5 of the same sum over absolute values."""
import numpy as np
import pytest
import torch

from tests.gpu_helpers import np_

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _bf16(a):
    return torch.as_tensor(np.asarray(a, np.float32)).to(torch.bfloat16)


def _act(gs, t):
    return gs.Act(t.to(DEV).contiguous())


WGRAD_CASES = [
    # (n, h, w, cin1, cin2, cout, masked)
    (1, 1, 1, 8, 0, 8, True),
    (1, 4, 32, 32, 0, 32, True),        # one step of one strip at 64 output channels
    (2, 5, 33, 32, 0, 64, True),        # a row and a column past them
    (1, 8, 31, 32, 0, 32, False),       # one step at 32
    (3, 9, 65, 64, 32, 32, True),       # three strips, an odd number of channel groups
    (1, 70, 40, 64, 0, 128, True),      # many steps per run
    (2, 13, 34, 128, 64, 64, True),
    (1, 6, 50, 40, 24, 72, False),      # groups cut short on both sides
    (1, 3, 7, 24, 0, 40, True),
    (9, 16, 96, 64, 64, 64, True),      # runs that cross strips and images
]


@pytest.mark.parametrize("case", WGRAD_CASES)
def test_wgrad_edges(gs, case):
    print(case, flush=True)
    n, h, w, c1, c2, cout, masked = case
    rng = np.random.default_rng(sum(case))
    x = _bf16(rng.normal(size=(n, h, w, c1 + c2)))
    y = _bf16(np.where(rng.random((n, h, w, cout)) < 0.1, -0.0, np.maximum(rng.normal(size=(n, h, w, cout)), 0.0)))
    # the gradient is a channel slice of a wider tensor
    wide = _bf16(rng.normal(size=(n, h, w, cout + 16)))
    gy = wide[..., 8:8 + cout]
    dw = torch.ones(9, cout, c1 + c2, device=DEV)
    db = torch.ones(cout, device=DEV)
    xa = _act(gs, x[..., :c1])
    xb = _act(gs, x[..., c1:]) if c2 else None
    gact = gs.Act(wide.to(DEV), cout, 8)
    gs.gs_nn_conv3x3_wgrad(xa, xb, gact, _act(gs, y) if masked else None, dw, db)
    only = torch.ones_like(dw)
    gs.gs_nn_conv3x3_wgrad(xa, xb, gact, _act(gs, y) if masked else None, only, None)
    torch.cuda.synchronize()
    dz = gy.double() * ((y > 0).double() if masked else 1.0)
    pad = torch.nn.functional.pad(x.double(), (0, 0, 1, 1, 1, 1))
    flat = dz.reshape(-1, cout)
    for k in range(9):
        tap = pad[:, k // 3:k // 3 + h, k % 3:k % 3 + w].reshape(-1, c1 + c2)
        ref, scale = flat.T @ tap + 1.0, flat.abs().T @ tap.abs() + 1.0
        for got in (dw, only):
            assert (np.abs(np_(got[k]) - ref.numpy()) <= 1e-5 * scale.numpy() + 1e-7).all(), (case, k)
    assert (np.abs(np_(db) - (flat.sum(0) + 1.0).numpy()) <= 1e-5 * (flat.abs().sum(0) + 1.0).numpy()).all()
