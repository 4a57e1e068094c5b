"""Results that are stored, and inputs that are loaded, with or without the non-temporal hint by their size: either way the same bits, and nothing
outside an output is written.  A call on one side of a line is compared with calls on parts of the same data, which lie on the other."""
import pytest
import torch

from tests.test_gpu_parity import M  # noqa: F401
from tests.test_gpu_row_blocks import between, untouched

pytestmark = pytest.mark.gpu


# (H, rows, cols) of a part; the whole is `parts` of them.  A whole and its parts lie on different sides of a line (or, the last of each kind, the count is ragged):
# binary32 rows of up to 256 elements are kept from 30 to 100 MB, 16-bit rows that start anywhere, beyond 256, from 30 to 75 MB, rows of 8k elements beyond 256 up to 180 MB
# (45 MB beyond 1024), of a multiple of 128 from 768 on from 30 to 45 MB
F32_ROWS = [(2, 9512, 197, 4), (3, 25008, 49, 6), (2, 38072, 197, 2), (1, 45685, 197, 1)]
LONG_ROWS = [(2, 8664, 577, 2), (1, 33264, 1127, 2), (1, 38403, 391, 1), (1, 57181, 577, 1)]
WAVE_ROWS = [(2, 113640, 264, 2), (1, 30000, 1000, 4), (2, 5000, 1616, 2), (2, 6512, 768, 2), (1, 10008, 2048, 2), (1, 4883, 3072, 2)]


def keeps(cols, size, dtype):
    eb = dtype.itemsize
    if cols <= 256:
        return eb == 4 and 30e6 <= size <= 100e6
    if cols % 8:
        return eb == 2 and 30e6 <= size <= 75e6
    return (cols >= 768 and 30e6 <= size <= 45e6) if cols % 128 == 0 else size <= (45e6 if cols > 1024 else 180e6)


@pytest.mark.parametrize("dtype,H,rows,cols,parts", [(torch.float32, *c) for c in F32_ROWS] + [(t, *c) for c in LONG_ROWS + WAVE_ROWS for t in (torch.float16, torch.bfloat16)])
def test_softmax_backward_kept_or_not(M, H, rows, cols, parts, dtype):  # noqa: F811
    """a call against calls on parts of the same data, and in place; a ragged whole against quarters of its rows"""
    size = parts * H * rows * cols * dtype.itemsize
    if parts > 1:
        assert keeps(cols, size, dtype) != keeps(cols, size // parts, dtype)
    else:
        assert keeps(cols, size, dtype) and H * rows * cols % 8
    g = torch.Generator(device="cuda").manual_seed(cols)
    q = torch.randint(-128, 128, (parts, H, rows, cols), dtype=torch.int8, device="cuda", generator=g)
    a, b = torch.rand(H, device="cuda", generator=g) + 0.1, torch.rand(H, device="cuda", generator=g)
    dy = torch.randn((parts, H, rows, cols), dtype=dtype, device="cuda", generator=g)
    out, dx = between(dy)
    M.mesa_softmax_bwd_q(q, parts, H, rows, cols, a, b, dy, dx)
    assert untouched(out)
    for k in range(parts if parts > 1 else 0):
        one, part = between(dy[k])
        M.mesa_softmax_bwd_q(q[k], 1, H, rows, cols, a, b, dy[k], part)
        assert untouched(one) and torch.equal(part, dx[k])
    if parts == 1:                                  # a quarter of the rows at a time, below the line
        cut = rows // 32 * 8
        for r in range(0, 4 * cut, cut):
            yq, d = q[0, 0, r:r + cut].clone(), dy[0, 0, r:r + cut].clone()
            assert not keeps(cols, d.numel() * dtype.itemsize, dtype)
            one, part = between(d)
            M.mesa_softmax_bwd_q(yq, 1, 1, cut, cols, a, b, d, part)
            assert untouched(one) and torch.equal(part, dx[0, 0, r:r + cut])
    M.mesa_softmax_bwd_q(q, parts, H, rows, cols, a, b, dy, dy)
    assert torch.equal(dy, dx)


# kept from 18 MB on, up to 80 MB in 16 bits and 120 MB in binary32: the whole beyond the upper line and its half below it, the half beyond the lower line and its half below that
@pytest.mark.parametrize("outer,groups,inner,dtype", [(30000, 12, 128, torch.float16), (9000, 3, 2401, torch.float16), (300, 6, 38809, torch.bfloat16), (30000, 12, 128, torch.float32),
                                                      (8000, 12, 128, torch.float16), (120, 3, 38809, torch.bfloat16), (4000, 12, 128, torch.float32), (2400, 3, 2401, torch.float16)])
def test_running_estimates_kept_or_not(M, outer, groups, inner, dtype):  # noqa: F811
    """a tensor and its half, on either side of a line, against torch's extrema"""
    g = torch.Generator(device="cuda").manual_seed(outer)
    x = torch.randn((outer, groups, inner), dtype=dtype, device="cuda", generator=g)
    low, high = 18000000, 120000000 if dtype == torch.float32 else 80000000
    size = [t.numel() * t.element_size() for t in (x, x[:outer // 2])]
    assert any(size[1] < line < size[0] for line in (low, high))
    for t in (x, x[:outer // 2]):
        n = (t.shape[0], groups, inner)
        ws = torch.empty(max(16, M.workspace_bytes(M.OP_UPDATE_RUNNING_PARAMS, *n)), dtype=torch.uint8, device="cuda")
        a, b = torch.zeros(groups, device="cuda"), torch.zeros(groups, device="cuda")
        M.mesa_update_running_params(t, n, a, b, 0.9, True, ws)
        lo, hi = t.amin(dim=(0, 2)).float(), t.amax(dim=(0, 2)).float()
        assert torch.equal(b, lo) and torch.equal(a, hi - lo)


# rows on half lines and of a multiple of 128 elements on either side of the lines of dA by tiles, every head size; all of them, and their halves, go by tiles
@pytest.mark.parametrize("heads,N,Dh", [(512, 96, 64), (640, 160, 32), (360, 288, 64), (3200, 128, 64), (600, 384, 96), (240, 480, 64), (70, 1056, 128), (100, 1024, 128), (24, 2176, 64), (12, 3712, 32)])
def test_attention_map_gradient_kept_or_not(M, heads, N, Dh):  # noqa: F811
    """Against float64: v^ and the result are each rounded to 16 bits (2^-11), so 2e-3 of the largest; against half as many heads, which take the same kernel, bit for bit."""
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
    assert untouched(one) and torch.equal(part, dA[half:])
