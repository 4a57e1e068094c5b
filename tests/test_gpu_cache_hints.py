"""Results that are stored, and inputs that are loaded, with or without the non-temporal hint by their size: either way the same bits, and nothing
outside an output is written.  A call on one side of a line is compared with calls on parts of the same data, which lie on the other."""
import pytest
import torch

from tests.test_gpu_parity import M  # noqa: F401
from tests.test_gpu_row_blocks import between, untouched

pytestmark = pytest.mark.gpu


# rows of 8k elements: up to 180 MB kept (from 30 MB on at multiples of 128); other rows from 30 to 100 MB
@pytest.mark.parametrize("dtype", [torch.float16, torch.float32], ids=["f16", "f32"])
@pytest.mark.parametrize("cols,whole_mb,part_mb", [(197, 60, 15), (197, 120, 60), (49, 40, 20), (577, 60, 20), (264, 240, 120), (512, 60, 15), (1616, 200, 100)])
def test_softmax_backward_kept_or_not(M, cols, whole_mb, part_mb, dtype):  # noqa: F811
    H, eb = 2, torch.empty(0, dtype=dtype).element_size()
    parts = whole_mb // part_mb
    rows = part_mb * 1000000 // (eb * H * cols) // 8 * 8
    g = torch.Generator(device="cuda").manual_seed(cols)
    q = torch.randint(-128, 128, (parts, H, rows, cols), dtype=torch.int8, device="cuda", generator=g)
    a, b = torch.rand(H, device="cuda", generator=g) + 0.1, torch.rand(H, device="cuda", generator=g)
    dy = torch.randn((parts, H, rows, cols), dtype=dtype, device="cuda", generator=g)
    out, dx = between(dy)
    M.mesa_softmax_bwd_q(q, parts, H, rows, cols, a, b, dy, dx)
    assert untouched(out)
    for k in range(parts):
        one, part = between(dy[k])
        M.mesa_softmax_bwd_q(q[k], 1, H, rows, cols, a, b, dy[k], part)
        assert untouched(one) and torch.equal(part, dx[k])


# kept from 18 MB on, up to 75 MB in 16 bits and 120 MB in binary32: the whole beyond the upper line and its half below it, the half beyond the lower line and its half below that
@pytest.mark.parametrize("outer,groups,inner,dtype", [(30000, 12, 128, torch.float16), (9000, 3, 2401, torch.float16), (300, 6, 38809, torch.bfloat16), (30000, 12, 128, torch.float32),
                                                      (8000, 12, 128, torch.float16), (120, 3, 38809, torch.bfloat16), (4000, 12, 128, torch.float32), (2400, 3, 2401, torch.float16)])
def test_running_estimates_kept_or_not(M, outer, groups, inner, dtype):  # noqa: F811
    """a tensor and its half, on either side of a line, against torch's extrema"""
    g = torch.Generator(device="cuda").manual_seed(outer)
    x = torch.randn((outer, groups, inner), dtype=dtype, device="cuda", generator=g)
    low, high = 18000000, 120000000 if dtype == torch.float32 else 75000000
    size = [t.numel() * t.element_size() for t in (x, x[:outer // 2])]
    assert any(size[1] < line < size[0] for line in (low, high))
    for t in (x, x[:outer // 2]):
        n = (t.shape[0], groups, inner)
        ws = torch.empty(max(16, M.workspace_bytes(M.OP_UPDATE_RUNNING_PARAMS, *n)), dtype=torch.uint8, device="cuda")
        a, b = torch.zeros(groups, device="cuda"), torch.zeros(groups, device="cuda")
        M.mesa_update_running_params(t, n, a, b, 0.9, True, ws)
        lo, hi = t.amin(dim=(0, 2)).float(), t.amax(dim=(0, 2)).float()
        assert torch.equal(b, lo) and torch.equal(a, hi - lo)


@pytest.mark.parametrize("heads,N,Dh", [(200, 96, 64), (150, 160, 32), (160, 288, 64), (24, 2176, 64), (8, 3712, 32)])
def test_attention_map_gradient_kept_or_not(M, heads, N, Dh):  # noqa: F811
    """dA by tiles: rows on half lines, and rows of a multiple of 128 elements on either side of 10^8 of them.  Against float64: v^ and the result are each
    rounded to 16 bits (2^-11), so 2e-3 of the largest; against half as many heads, which may take the general kernel, one unit of the result (2^-10)."""
    g = torch.Generator(device="cuda").manual_seed(N)
    code = lambda n: torch.randint(-128, 128, (heads, n, Dh), dtype=torch.int8, device="cuda", generator=g)  # noqa: E731
    aq, vq = torch.randint(-128, 128, (heads, N, N), dtype=torch.int8, device="cuda", generator=g), code(N)
    s, o = torch.rand(1, device="cuda", generator=g) + 0.1, torch.rand(1, device="cuda", generator=g)
    dO = torch.randn((heads, N, Dh), dtype=torch.float16, device="cuda", generator=g)
    (out, dA), dV = between(torch.empty((heads, N, N), dtype=torch.float16)), torch.empty_like(dO)
    M.mesa_attn_av_bwd_q(aq, vq, heads, 1, N, Dh, s, o, s, o, dO, dA, dV)
    assert untouched(out)
    v_hat = (vq.float() + 128) * (s / 255) + o
    for k in range(0, heads, max(1, heads // 8)):
        ref = dO[k].double() @ v_hat[k].double().t().contiguous()
        assert float((dA[k].double() - ref).abs().max() / ref.abs().max()) <= 2e-3
    half = heads // 2
    (one, part), dV = between(torch.empty((half, N, N), dtype=torch.float16)), torch.empty_like(dO[:half])
    M.mesa_attn_av_bwd_q(aq[half:], vq[half:], half, 1, N, Dh, s, o, s, o, dO[half:], part, dV)
    assert untouched(one)
    diff = (part.float() - dA[half:].float()).abs().max() / dA.float().abs().max()
    assert float(diff) <= 2 ** -10
