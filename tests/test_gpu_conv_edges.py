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
    (1, 33, 70, 768, 0, 800, True),     # enough work for 64 x 64 channels a workgroup
    (2, 30, 40, 712, 24, 776, True),    # and for 64 x 32
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


CONV_CASES = [
    # (n, h, w, cin1, cin2, cout, masked, channel offset of the output)
    (1, 1, 1, 8, 0, 8, False, 0),
    (1, 16, 16, 32, 0, 32, False, 0),      # exactly one tile
    (2, 17, 33, 32, 0, 32, True, 8),       # a row and a column past it, a channel slice
    (1, 5, 40, 64, 32, 32, False, 0),      # three chunks, concatenated
    (1, 20, 20, 32, 0, 96, True, 0),       # three groups of 32 channels
    (1, 18, 15, 24, 0, 72, True, 0),       # the third cut to 8
    (1, 9, 70, 32, 0, 65, False, 0),       # channel counts that are not multiples of 8:
    (1, 9, 30, 40, 0, 20, False, 0),       # element by element
    (1, 9, 30, 32, 0, 32, False, 3),       # and an output that is not 16-byte aligned
    (2, 30, 21, 128, 64, 64, True, 0),
    (3, 120, 160, 32, 0, 128, True, 0),    # four groups, more workgroups than places
]


@pytest.mark.parametrize("case", CONV_CASES)
def test_conv_edges(gs, case):
    print(case, flush=True)
    n, h, w, c1, c2, cout, masked, off = case
    cin = c1 + c2
    rng = np.random.default_rng(sum(case))
    x = _bf16(rng.normal(size=(n, h, w, cin)))
    m = _bf16(np.where(rng.random((n, h, w, cin)) < 0.1, -0.0, rng.normal(size=(n, h, w, cin))))
    wt = _bf16(rng.normal(size=(9, cout, cin)) / np.sqrt(9 * cin))
    b = torch.as_tensor(rng.normal(size=cout).astype(np.float32))
    stride = (cout + off + 7) // 8 * 8 + 8
    xa, xb = _act(gs, x[..., :c1]), _act(gs, x[..., c1:]) if c2 else None
    mask = _act(gs, m) if masked else None
    xm = x.double() * ((m > 0).double() if masked else 1.0)
    pad = torch.nn.functional.pad(xm, (0, 0, 1, 1, 1, 1))
    taps = [pad[:, k // 3:k // 3 + h, k % 3:k % 3 + w] for k in range(9)]
    ref = sum(t @ wt[k].double().T for k, t in enumerate(taps)) + b.double()
    scale = (sum(t.abs() @ wt[k].double().abs().T for k, t in enumerate(taps)) + b.double().abs()).numpy()
    for relu in (False, True):
        wide = torch.full((n, h, w, stride), -7.0, dtype=torch.bfloat16, device=DEV)
        yf = torch.full((n * h * w, cout + 3), -7.0, device=DEV)
        gs.gs_nn_conv3x3(xa, xb, mask, wt.to(DEV), cout, b.to(DEV), relu, gs.Act(wide, cout, off), yf, cout + 3)
        torch.cuda.synchronize()
        want = ref.clamp(min=0) if relu else ref
        got = np_(yf)[:, :cout].reshape(n, h, w, cout)
        assert (np.abs(got - want.numpy()) <= 1e-5 * scale + 1e-7).all(), case
        # the bf16 output is the rounding of the float32 one, and nothing beside it is written
        assert torch.equal(wide[..., off:off + cout].reshape(-1, cout), yf[:, :cout].to(torch.bfloat16))
        assert (wide[..., :off] == -7).all() and (wide[..., off + cout:] == -7).all()
        assert (yf[:, cout:] == -7).all()


@pytest.mark.parametrize("case", [(2, 9, 40, 32, 32), (1, 12, 31, 32, 32), (1, 16, 33, 64, 32),
                                  (2, 7, 40, 64, 64), (1, 33, 70, 768, 768), (2, 30, 40, 736, 776)])
def test_wgrad_infinite_inputs_at_the_image_edge(gs, case):
    """The input's last row and column are infinite in a channel each: a tap that never
    reads one of them stays finite there, with the strip's or the step's end in the image
    and beyond it, in each of the kernel's three widths."""
    print(case, flush=True)
    n, h, w, cin, cout = case
    rng = np.random.default_rng(sum(case))
    x = _bf16(rng.normal(size=(n, h, w, cin)))
    x[:, h - 1, :, 0] = np.inf
    x[:, :, w - 1, 1] = np.inf
    gy = _bf16(rng.normal(size=(n, h, w, cout)))
    gy[gy == 0] = 1.0
    dw = torch.zeros(9, cout, cin, device=DEV)
    gs.gs_nn_conv3x3_wgrad(_act(gs, x), None, _act(gs, gy), None, dw, None)
    torch.cuda.synchronize()
    for k in range(9):
        dy, dx = k // 3 - 1, k % 3 - 1   # pixels (y, x) whose neighbour (y + dy, x + dx) lies in the image
        own = gy.double()[:, max(0, -dy):h - max(0, dy), max(0, -dx):w - max(0, dx)].reshape(-1, cout)
        tap = x.double()[:, max(0, dy):h + min(0, dy), max(0, dx):w + min(0, dx)].reshape(-1, cin)
        finite = torch.isfinite(tap).all(0)
        assert finite[2:].all() and bool(finite[0]) == (dy < 0) and bool(finite[1]) == (dx < 0)
        got, ref, scale = dw[k].cpu(), own.T @ tap, own.abs().T @ tap.abs()
        err = (got - ref).abs()[:, finite]
        assert (err <= 1e-5 * scale[:, finite] + 1e-7).all(), (case, k)
        assert not torch.isfinite(got[:, ~finite]).any(), (case, k)


# 16 x 16 tiles times 64-channel groups from 1,024 on, where a workgroup takes 64 channels
WIDE_CONV_CASES = [
    # (n, h, w, cin1, cin2, cout, masked, channel offset of the output)
    (1, 512, 512, 64, 0, 64, True, 8),      # exactly 1,024, whole tiles
    (1, 512, 496, 64, 0, 64, True, 8),      # 992: 32 channels at a time
    (2, 330, 250, 64, 32, 128, True, 0),    # cut tiles, three chunks, concatenated
    (2, 330, 250, 64, 32, 128, False, 8),
    (1, 250, 260, 128, 0, 200, True, 0),    # the last group cut to 8 channels
    (1, 250, 260, 120, 0, 200, False, 0),   # and the last chunk to 24
    (1, 520, 260, 32, 0, 65, False, 0),     # one chunk; element by element
    (1, 520, 260, 40, 0, 128, True, 3),     # an output that is not 16-byte aligned
]


@pytest.mark.parametrize("case", WIDE_CONV_CASES)
def test_conv_64_channels_a_workgroup(gs, case):
    print(case, flush=True)
    n, h, w, c1, c2, cout, masked, off = case
    cin = c1 + c2
    gen = torch.Generator(device=DEV).manual_seed(sum(case))
    rand = lambda *s: torch.randn(*s, generator=gen, device=DEV)
    x = rand(n, h, w, cin).to(torch.bfloat16)
    m = rand(n, h, w, cin)
    m = torch.where(rand(n, h, w, cin) < -1.3, torch.full_like(m, -0.0), m).to(torch.bfloat16)
    wt = (rand(9, cout, cin) / (9 * cin) ** 0.5).to(torch.bfloat16)
    b = rand(cout)
    stride = (cout + off + 7) // 8 * 8 + 8
    xa, xb = _act(gs, x[..., :c1]), _act(gs, x[..., c1:]) if c2 else None
    wide = torch.full((n, h, w, stride), -7.0, dtype=torch.bfloat16, device=DEV)
    yf = torch.full((n * h * w, cout + 3), -7.0, device=DEV)
    gs.gs_nn_conv3x3(xa, xb, _act(gs, m) if masked else None, wt, cout, b, True, gs.Act(wide, cout, off), yf, cout + 3)
    torch.cuda.synchronize()
    xm = x.double() * ((m > 0).double() if masked else 1.0)
    pad = torch.nn.functional.pad(xm, (0, 0, 1, 1, 1, 1))
    ref = b.double().expand(n * h * w, cout).clone()
    scale = ref.abs()
    for k in range(9):
        tap = pad[:, k // 3:k // 3 + h, k % 3:k % 3 + w].reshape(-1, cin)
        wk = wt[k].double().T.contiguous()
        ref += tap @ wk
        scale += tap.abs() @ wk.abs()
    got = yf[:, :cout]
    assert bool(((got - ref.clamp(min=0)).abs() <= 1e-5 * scale + 1e-7).all()), case
    assert torch.equal(wide[..., off:off + cout].reshape(-1, cout), got.to(torch.bfloat16))
    assert (wide[..., :off] == -7).all() and (wide[..., off + cout:] == -7).all()
    assert (yf[:, cout:] == -7).all()
