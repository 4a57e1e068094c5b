"""Softmax forward and backward over rows longer than 256 elements: the kernels that keep a tile of unaligned rows in LDS and
the one that keeps an aligned row in a wave's registers, at the edges of their shapes, against the CPU oracle.

Bounds: those of the other softmax tests (1e-5, 2e-3, 1.6e-2 of the largest result by storage type); codes and running
estimates bit for bit on the stored map.
"""
import numpy as np
import pytest
import torch

from oracle import mesa_ref as R
from tests.test_gpu_parity import DTYPE_IDS, DTYPES, TOL, _mid_of_frame, npy, relerr, ws_for

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def M():
    import paper_2111_11124_amd as m
    assert torch.cuda.is_available(), "these tests need the MI355X"
    m.lib()
    return m


# unaligned: both ends of every slot count, one, two and four rows to a vector boundary; aligned: both ends of every lane
# group.  Maps of one, three and seven rows put several heads into a tile, the odd row counts leave a ragged last one.
SHAPES = [(1, 2, 3, 257), (1, 3, 7, 258), (2, 3, 5, 260), (1, 2, 9, 383), (1, 2, 9, 385), (1, 1, 17, 511), (1, 2, 9, 513), (1, 3, 11, 577),
          (1, 2, 5, 641), (1, 5, 1, 700), (1, 2, 9, 769), (2, 1, 7, 1023), (1, 2, 5, 1025), (1, 2, 3, 1281), (1, 1, 9, 1537), (1, 1, 8, 2046),
          (1, 1, 9, 2047),
          (1, 3, 5, 264), (1, 2, 7, 384), (1, 2, 6, 392), (1, 2, 5, 512), (1, 3, 3, 520), (1, 1, 7, 768), (1, 2, 3, 776), (1, 1, 5, 1024), (1, 1, 3, 1032),
          (1, 1, 5, 1536), (1, 1, 3, 2048), (1, 1, 3, 2056), (1, 1, 2, 3080), (1, 1, 3, 4096)]


def _params(H, g):
    return 0.05 + 0.2 * torch.rand(H, device="cuda", generator=g), 0.01 * torch.rand(H, device="cuda", generator=g)


@pytest.mark.parametrize("dtype", DTYPES, ids=DTYPE_IDS)
@pytest.mark.parametrize("B,H,rows,cols", SHAPES)
def test_softmax_backward_long_rows(M, B, H, rows, cols, dtype):
    g = torch.Generator(device="cuda").manual_seed(rows * 5000 + cols)
    n = B * H * rows * cols
    q = _mid_of_frame(torch.randint(-128, 128, (n,), dtype=torch.int8, device="cuda", generator=g), 127)
    dy = _mid_of_frame(torch.randn(n, device="cuda", generator=g).to(dtype), float("nan"))
    a, b = _params(H, g)
    out = torch.full((n + 128,), 7.0, dtype=dtype, device="cuda")
    M.mesa_softmax_bwd_q(q, B, H, rows, cols, a, b, dy, out[64:64 + n])
    ref = R.softmax_bwd_q(npy(q), B, H, rows, cols, npy(a), npy(b), npy(dy))
    got = npy(out)
    assert np.all(got[:64] == 7) and np.all(got[64 + n:] == 7)
    assert relerr(got[64:64 + n].reshape(np.shape(ref)), ref) <= TOL[dtype]
    M.mesa_softmax_bwd_q(q, B, H, rows, cols, a, b, dy, dy)       # in place
    assert np.array_equal(npy(dy), got[64:64 + n])


@pytest.mark.parametrize("dtype", DTYPES, ids=DTYPE_IDS)
@pytest.mark.parametrize("B,H,rows,cols", [s for s in SHAPES if s[3] % 8])
def test_softmax_forward_long_rows(M, B, H, rows, cols, dtype):
    """Masked logits among them: -infinity, and rows of nothing but the type's lowest value, which come out even."""
    g = torch.Generator(device="cuda").manual_seed(rows * 7000 + cols)
    n = B * H * rows * cols
    s = torch.randn((B, H, rows, cols), device="cuda", generator=g) * 3
    s[torch.rand(s.shape, device="cuda", generator=g) < 0.1] = -float("inf")
    s = s.to(dtype)
    s[0, 0, rows - 1] = torch.finfo(dtype).min
    s = _mid_of_frame(s, float("nan"))
    ws = ws_for(M, M.OP_SOFTMAX_FWD_Q, B * H * rows, H, cols, dtype)
    for mode in (M.ROUND_STOCHASTIC, M.ROUND_NEAREST_EVEN):
        a, b = _params(H, torch.Generator(device="cuda").manual_seed(5))
        a0, b0 = npy(a).copy(), npy(b).copy()
        y = torch.full((n + 128,), 7.0, dtype=dtype, device="cuda")
        q = torch.full((n + 128,), 99, dtype=torch.int8, device="cuda")
        M.mesa_softmax_fwd_q(s, B, H, rows, cols, a, b, 0.9, y[64:64 + n], q[64:64 + n], ws, mode, 77, 1000)
        ref = R.softmax_fwd(npy(s), B * H * rows, cols)
        got = npy(y)
        assert np.all(got[:64] == 7) and np.all(got[64 + n:] == 7) and torch.all(q[:64] == 99) and torch.all(q[64 + n:] == 99)
        assert relerr(got[64:64 + n].reshape(np.shape(ref)), ref) <= TOL[dtype]
        rq, ra, rb = R.quantize_update_fused(got[64:64 + n].copy(), (B, H, rows * cols), a0, b0, 0.9, mode, 77, 1000)
        assert np.array_equal(npy(q)[64:64 + n], rq.reshape(-1))
        assert np.array_equal(npy(a), ra) and np.array_equal(npy(b) + np.float32(0), rb + np.float32(0))


@pytest.mark.parametrize("dtype", DTYPES, ids=DTYPE_IDS)
@pytest.mark.parametrize("cols", [577, 1023])
def test_softmax_forward_long_rows_in_the_smallest_workspace(M, cols, dtype):
    """Room for the extrema of fewer workgroups than a resident round -- what the tiled kernel's 768 need is accepted: fewer
    workgroups that take several tiles each, the same bits."""
    B, H, rows = 16, 12, 577
    g = torch.Generator(device="cuda").manual_seed(3)
    s = torch.randn((B, H, rows, cols), device="cuda", generator=g).to(dtype)
    full = ws_for(M, M.OP_SOFTMAX_FWD_Q, B * H * rows, H, cols, dtype)
    least = 768 * 2 * H * 4 + 16
    assert full.numel() >= 1024 * 2 * H * 4 + 16            # a resident round is more than that
    got = []
    for ws in (full, full[:least]):
        a, b = torch.full((H,), 0.1, device="cuda"), torch.zeros(H, device="cuda")
        y, q = torch.empty_like(s), torch.empty(s.numel(), dtype=torch.int8, device="cuda")
        M.mesa_softmax_fwd_q(s, B, H, rows, cols, a, b, 0.9, y, q, ws, M.ROUND_STOCHASTIC, 9, 0)
        got.append((y, q, a, b))
    for u, v in zip(*got):
        assert torch.equal(u, v)
    with pytest.raises(M.MesaError) as e:
        M.mesa_softmax_fwd_q(s, B, H, rows, cols, a, b, 0.9, y, q, full[:least - 16], M.ROUND_STOCHASTIC, 9, 0)
    assert e.value.status == M.ERR_WORKSPACE


@pytest.mark.parametrize("dtype", DTYPES, ids=DTYPE_IDS)
@pytest.mark.parametrize("cols", [257, 577, 1000, 1023, 1127, 2047, 2050])
def test_softmax_backward_long_rows_near_the_smallest_value(M, cols, dtype):
    """Nearly every element of a long attention map has the smallest codes, and its map's offset is orders of magnitude below the
    range: x_bar * alpha / 255 + beta is rounded once, element by element, not taken off a number of the range's size.
    Bound: a unit of the type (the result is rounded to it once, the arithmetic before is binary32) and, for d, 1e-6 of the terms
    that it adds."""
    H, rows = 2, 24
    n = H * rows * cols
    g = torch.Generator(device="cuda").manual_seed(cols)
    q = torch.full((n,), -128, dtype=torch.int8, device="cuda")
    few = torch.rand(n, device="cuda", generator=g) < 0.02
    q[few] = torch.randint(-128, 128, (int(few.sum()),), dtype=torch.int8, device="cuda", generator=g)
    dy = (torch.randn(n, device="cuda", generator=g) * 4096).to(dtype)
    a, b = torch.tensor([0.06, 0.9], device="cuda"), torch.tensor([3e-6, 1e-5], device="cuda")
    dx = torch.empty(n, dtype=dtype, device="cuda")
    M.mesa_softmax_bwd_q(q, 1, H, rows, cols, a, b, dy, dx)
    y = (q.double().view(H, rows, cols) + 128) * (a.double() / 255).view(H, 1, 1) + b.double().view(H, 1, 1)
    gy = dy.double().view(H, rows, cols)
    d = (gy * y).sum(-1, keepdim=True)
    ref = y * (gy - d)
    slack = y * 1e-6 * ((gy * y).abs().sum(-1, keepdim=True) + gy.abs())
    unit = 0.5 * torch.finfo(dtype).eps + 2.0 ** -21
    least = {torch.float32: 2.0 ** -149, torch.float16: 2.0 ** -24, torch.bfloat16: 2.0 ** -133}[dtype]
    assert ((dx.double().view(H, rows, cols) - ref).abs() <= unit * ref.abs() + slack + least).all()


@pytest.mark.parametrize("cols", [384, 512])
def test_softmax_backward_long_rows_sums_a_row_in_short_chains(M, cols):
    """binary32, even rows, a gradient of 100 with noise of 1: what is left of dy - d is 100 times smaller than the terms that d is the
    sum of.  A sum of all in a balanced tree is off by 3.1e-6 (2^-17 sqrt(1/12) for the last addition, half a square less for
    each level before); vectors of eight and four of them to a lane before the tree: under 3.9e-6, one chain of all: above."""
    H, rows = 4, 2048
    n = H * rows * cols
    g = torch.Generator(device="cuda").manual_seed(1)
    y = torch.softmax(torch.randn((H, rows, cols), device="cuda", generator=g).double(), -1)
    a, b = y.amax((1, 2)).float(), torch.zeros(H, device="cuda")
    q = (y / a.double().view(H, 1, 1) * 255).round().clamp(0, 255).sub(128).to(torch.int8).contiguous()
    dy = torch.randn(n, device="cuda", generator=g) + 100
    dx = torch.empty(n, device="cuda")
    M.mesa_softmax_bwd_q(q, 1, H, rows, cols, a, b, dy, dx)
    yh, gy = (q.double() + 128) * (a.double() / 255).view(H, 1, 1), dy.double().view(H, rows, cols)
    ref = yh * (gy - (gy * yh).sum(-1, keepdim=True))
    assert (dx.double().view(H, rows, cols) - ref).norm() <= 3.9e-6 * ref.norm()
