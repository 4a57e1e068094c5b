"""The binary32 products at de-quantized operands over the whole range of binary32: values whose last bits are subnormal,
subnormal values, and values too large for the matrix cores' bfloat16 parts, column by column (or head by head) on its
own scale.  Reference: the definition in binary64.

Bound: 1e-5 of the column's (head's) largest result, the binary32 bound of the other tests, and where results are subnormal a
unit of 2^-149 for each rounding of a sum: two at the end and one per slice of at least 64 rows."""
import pytest
import torch

pytestmark = pytest.mark.gpu

EXPONENTS = [0, -60, -100, -103, -104, -110, -116, -122, -126, -127, -130, -136, -142, -148, 40, 60, 61, 62, 63, 66, 90, 105]


@pytest.fixture(scope="module")
def M():
    import paper_2111_11124_amd as m
    assert torch.cuda.is_available(), "these tests need the MI355X"
    m.lib()
    return m


def _scaled(t, dim, exponents):
    """t times 2^e along dim, rounded once to binary32"""
    shape = [1] * t.dim()
    shape[dim] = t.shape[dim]
    e = torch.tensor([exponents[i % len(exponents)] for i in range(t.shape[dim])], dtype=torch.float64, device=t.device)
    return (t.double() * torch.exp2(e).view(shape)).float()


def _check(got, ref, dim, roundings):
    dims = [d for d in range(ref.dim()) if d != dim]
    err, top = (got.double() - ref).abs().amax(dims), ref.abs().amax(dims)
    assert torch.isfinite(got).all()
    bad = err > 1e-5 * top + roundings * 2.0 ** -149
    assert not bad.any(), [(i, EXPONENTS[i % len(EXPONENTS)], (err[i] / top[i]).item()) for i in bad.nonzero().flatten().tolist()]


@pytest.mark.parametrize("exponents", [EXPONENTS, [e for e in EXPONENTS if e < 60]], ids=["with-large", "cut"])
@pytest.mark.parametrize("Mr,K,N", [(1, 16, 44), (33, 48, 44), (70, 144, 132), (500, 96, 72), (4099, 80, 136)])
def test_linear_dw_over_the_range_of_binary32(M, Mr, K, N, exponents):
    g = torch.Generator(device="cuda").manual_seed(Mr + K)
    q = torch.randint(-128, 128, (Mr, K), dtype=torch.int8, device="cuda", generator=g)
    dy = _scaled(torch.randn((Mr, N), device="cuda", generator=g), 1, exponents)
    a, b = torch.full((1,), 0.7, device="cuda"), torch.full((1,), -0.2, device="cuda")
    ws = torch.empty(M.workspace_bytes(M.OP_LINEAR_DW_Q, Mr, K, N, M.F32), dtype=torch.uint8, device="cuda")
    dW, db = torch.empty((N, K), device="cuda"), torch.empty(N, device="cuda")
    M.mesa_linear_dw_q(q, Mr, K, 1, a, b, dy, N, dW, db, ws)
    x_hat = (q.double() + 128) * (a.double() / 255) + b.double()
    ref = dy.double().t().contiguous() @ x_hat
    for r0 in range(0, N, len(exponents)):                       # rows of dW are columns of dy
        _check(dW[r0:r0 + len(exponents)], ref[r0:r0 + len(exponents)], 0, 2 + Mr // 64)


@pytest.mark.parametrize("N,Dh", [(33, 40), (64, 64), (197, 64), (300, 33)])
def test_attention_products_over_the_range_of_binary32(M, N, Dh):
    B, H = 1, len(EXPONENTS)
    g = torch.Generator(device="cuda").manual_seed(N)

    def codes(*shape):
        return torch.randint(-128, 128, shape, dtype=torch.int8, device="cuda", generator=g)

    A, V, Q, K = codes(B, H, N, N), codes(B, H, N, Dh), codes(B, H, N, Dh), codes(B, H, N, Dh)
    a, b = torch.full((H,), 0.7, device="cuda"), torch.full((H,), -0.2, device="cuda")
    dO, dS = (_scaled(torch.randn(s, device="cuda", generator=g), 1, EXPONENTS) for s in ((B, H, N, Dh), (B, H, N, N)))
    dA, (dV, dQ, dK) = torch.empty((B, H, N, N), device="cuda"), (torch.empty((B, H, N, Dh), device="cuda") for _ in range(3))
    M.mesa_attn_av_bwd_q(A, V, B, H, N, Dh, a, b, a, b, dO, dA, dV)
    M.mesa_attn_qk_bwd_q(Q, K, B, H, N, Dh, a, b, a, b, dS, 0.125, dQ, dK)
    hat = [((t.double() + 128) * (a[0].double() / 255) + b[0].double()).cpu() for t in (A, V, Q, K)]
    dO, dS = dO.double().cpu(), dS.double().cpu()
    for got, ref in ((dA, dO @ hat[1].transpose(-1, -2).contiguous()), (dV, hat[0].transpose(-1, -2).contiguous() @ dO),
                     (dQ, 0.125 * dS @ hat[3]), (dK, 0.125 * dS.transpose(-1, -2).contiguous() @ hat[2])):
        _check(got.cpu(), ref, 1, 2 + N // 64)


@pytest.mark.parametrize("at_nan,at_large", [(0, 1), (1, 0), (0, 2), (3, 1), (2, 3), (5, 4)])
def test_linear_dw_with_a_nan_beside_a_large_value(M, at_nan, at_large):
    """Both in one row of dy, in one thread's vector: the NaN stays in its row of dW and hides the large value from nobody."""
    Mr, K, N = 70, 48, 20
    g = torch.Generator(device="cuda").manual_seed(8 * at_nan + at_large)
    q = torch.randint(-128, 128, (Mr, K), dtype=torch.int8, device="cuda", generator=g)
    dy = torch.randn((Mr, N), device="cuda", generator=g)
    dy[33, at_nan], dy[33, at_large] = float("nan"), 1e33
    a, b = torch.full((1,), 0.7, device="cuda"), torch.full((1,), -0.2, device="cuda")
    ws = torch.empty(M.workspace_bytes(M.OP_LINEAR_DW_Q, Mr, K, N, M.F32), dtype=torch.uint8, device="cuda")
    dW, db = torch.empty((N, K), device="cuda"), torch.empty(N, device="cuda")
    M.mesa_linear_dw_q(q, Mr, K, 1, a, b, dy, N, dW, db, ws)
    ref = dy.double().t().contiguous() @ ((q.double() + 128) * (a.double() / 255) + b.double())
    assert torch.isnan(dW[at_nan]).all() and torch.isnan(db[at_nan])
    rest = torch.arange(N, device="cuda") != at_nan
    assert ((dW - ref)[rest].abs().amax(1) <= 1e-5 * ref[rest].abs().amax(1)).all()
