"""The weight gradient's tiles and slices: matrices on both sides of the line between the small and the large tiles, one slice
(whose workgroups finish dW themselves) and several, ragged in every extent.  Reference: the definition in binary64 on the
GPU (the CPU oracle would take minutes at these sizes; the two agree elsewhere)."""
import pytest
import torch

pytestmark = pytest.mark.gpu

# 2e-3 of the largest result: the bound of the 16-bit weight gradient tests (exact products, binary32 sums)
TOL = 2e-3


@pytest.fixture(scope="module")
def M():
    import paper_2111_11124_amd as m
    assert torch.cuda.is_available(), "these tests need the MI355X"
    m.lib()
    return m


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16], ids=["f16", "bf16"])
@pytest.mark.parametrize("Mr,K,N,G", [
    (50437, 768, 520, 3), (50437, 400, 1000, 1),          # beyond the line: 256 x 256 and 256 x 128 tiles, several slices
    (300, 8192, 8200, 8), (300, 1008, 65536, 1),          # and one slice
    (23451, 768, 1000, 3), (23400, 1008, 768, 3),         # below it, close to it
    (1, 16, 8, 1), (127, 112, 136, 1), (129, 128, 120, 2), (511, 1344, 1088, 6), (4097, 768, 264, 12)])
def test_linear_dw_tiles_and_slices(M, Mr, K, N, G, dtype):
    g = torch.Generator(device="cuda").manual_seed(Mr + K)
    q = torch.randint(-128, 128, (Mr, K), dtype=torch.int8, device="cuda", generator=g)
    dy = torch.randn((Mr, N), device="cuda", generator=g).to(dtype)
    a, b = 0.5 + torch.rand(G, device="cuda", generator=g), -torch.rand(G, device="cuda", generator=g)
    ws = torch.empty(M.workspace_bytes(M.OP_LINEAR_DW_Q, Mr, K, N, M.F16), dtype=torch.uint8, device="cuda")
    out = torch.full((N * K + 128,), 7.0, device="cuda")
    dW, db = out[64:64 + N * K].view(N, K), torch.empty(N, device="cuda")
    M.mesa_linear_dw_q(q, Mr, K, G, a, b, dy, N, dW, db, ws)
    x_hat = (q.double() + 128) * (a.double() / 255).repeat_interleave(K // G) + b.double().repeat_interleave(K // G)
    ref = dy.double().t().contiguous() @ x_hat
    assert (dW - ref).abs().max() <= TOL * ref.abs().max()
    assert (db - dy.double().sum(0)).abs().max() <= 1e-5 * dy.double().abs().sum(0).max()
    assert torch.all(out[:64] == 7) and torch.all(out[64 + N * K:] == 7)
    again = dW.clone()
    M.mesa_linear_dw_q(q, Mr, K, G, a, b, dy, N, dW, None, ws)      # without the bias gradient: the same bits
    assert torch.equal(dW, again)


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16], ids=["f16", "bf16"])
@pytest.mark.parametrize("Mr,K,N,G,sized_for", [(2961, 384, 384, 6, 3200), (1422, 384, 1152, 1, 1472), (2961, 384, 384, 6, None), (511, 1344, 1088, 6, 511),
                                                (4097, 768, 264, 12, 4097), (129, 128, 120, 2, 129)])
def test_linear_dw_of_small_matrices_in_the_workspace_there_is(M, Mr, K, N, G, sized_for, dtype):
    """The small tile in a workspace sized for more rows, which holds fewer slices than it would take, in one of a single slice (None)
    and in its own; matrices that k_dw_waves takes need none of it.  1e-5 of the largest result, the binary32 bound: every product is exact in binary32, and the sums are of
    centred codes or in short chains (contracting 1024 + code, as the large binary16 tiles do, misses it)."""
    g = torch.Generator(device="cuda").manual_seed(Mr + K)
    q = torch.randint(-128, 128, (Mr, K), dtype=torch.int8, device="cuda", generator=g)
    dy = torch.randn((Mr, N), device="cuda", generator=g).to(dtype)
    a, b = 0.5 + torch.rand(G, device="cuda", generator=g), -torch.rand(G, device="cuda", generator=g)
    one = (N * K + N) * 4 + 16
    need = M.workspace_bytes(M.OP_LINEAR_DW_Q, Mr, K, N, M.F16)
    n = M.workspace_bytes(M.OP_LINEAR_DW_Q, sized_for, K, N, M.F16) if sized_for else one
    assert n == need if sized_for == Mr else n < need
    frame = torch.full((n + 256,), 0x55, dtype=torch.uint8, device="cuda")
    dW, db = torch.empty((N, K), device="cuda"), torch.empty(N, device="cuda")
    M.mesa_linear_dw_q(q, Mr, K, G, a, b, dy, N, dW, db, frame[:n])
    x_hat = (q.double() + 128) * (a.double() / 255).repeat_interleave(K // G) + b.double().repeat_interleave(K // G)
    ref = dy.double().t().contiguous() @ x_hat
    assert (dW - ref).abs().max() <= 1e-5 * ref.abs().max()
    assert (db - dy.double().sum(0)).abs().max() <= 1e-5 * dy.double().abs().sum(0).max()
    assert torch.all(frame[n:] == 0x55)                     # nothing behind the workspace


@pytest.mark.parametrize("share", [1.0, 0.03], ids=["half-zero", "sparse"])
@pytest.mark.parametrize("Mr,K,N", [(394, 192, 768), (505, 1344, 1088), (2000, 2048, 1024), (4096, 768, 768), (12000, 768, 768), (25216, 1536, 384)])
def test_linear_dw_bfloat16_behind_a_rectifier(M, Mr, K, N, share):
    """Inputs of one sign, at least half of them zero and thus the smallest code, gradients with a mean.  Bound on the 2-norm, against
    the definition in binary64: a zero adds nothing, and a sum of terms of one sign is off by some 2^-25 of itself for
    the 16 roundings of a chain of 256 rows and for each chain and slice, at random: under 2e-7."""
    g = torch.Generator(device="cuda").manual_seed(Mr + K)
    x = torch.randn((Mr, K), device="cuda", generator=g).clamp(min=0)
    x[torch.rand((Mr, K), device="cuda", generator=g) >= share] = 0
    q = (x / 4 * 255).round().clamp(0, 255).sub(128).to(torch.int8)
    dy = (torch.randn((Mr, N), device="cuda", generator=g) + 0.5).bfloat16()
    a, b = torch.full((1,), 4.0, device="cuda"), torch.zeros(1, device="cuda")
    ws = torch.empty(M.workspace_bytes(M.OP_LINEAR_DW_Q, Mr, K, N, M.BF16), dtype=torch.uint8, device="cuda")
    dW, db = torch.empty((N, K), device="cuda"), torch.empty(N, device="cuda")
    M.mesa_linear_dw_q(q, Mr, K, 1, a, b, dy, N, dW, db, ws)
    ref = dy.double().t().contiguous() @ ((q.double() + 128) * (4.0 / 255))
    assert (dW - ref).norm() <= 2e-7 * ref.norm()
