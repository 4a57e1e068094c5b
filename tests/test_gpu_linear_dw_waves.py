"""The weight gradient of small matrices, a 32 x 32 tile per workgroup of sixteen or eight waves: rows around the waves' blocks of 32, ragged
tiles, both sides of the lines between the two and behind them.  Reference: the definition in binary64 on the GPU."""
import pytest
import torch

pytestmark = pytest.mark.gpu

# 1e-5 of the largest result, the binary32 bound: every product is exact in binary32 and the chains of sums are short
TOL = 1e-5


@pytest.fixture(scope="module")
def M():
    import paper_2111_11124_amd as m
    assert torch.cuda.is_available(), "these tests need the MI355X"
    m.lib()
    return m


# (only binary32 values are cut into parts, and those of 2^64 and more are not)
@pytest.mark.parametrize("dtype,largest", [(torch.float16, 1.0), (torch.bfloat16, 1.0), (torch.float32, 1.0), (torch.float32, 3e19)],
                         ids=["f16", "bf16", "f32", "f32 large"])
@pytest.mark.parametrize("Mr,K,N,G", [
    (1, 16, 8, 1), (31, 48, 40, 3), (33, 32, 32, 2), (481, 112, 136, 7), (512, 192, 64, 3), (513, 64, 200, 2),
    (2048, 80, 72, 5), (2049, 80, 72, 5),                                        # the most rows, and one more
    (197, 512, 512, 4), (197, 512, 520, 4), (255, 528, 8, 1), (257, 640, 1024, 5), (300, 640, 1032, 5)])   # 256 and 640 tiles, and more
def test_linear_dw_of_small_matrices(M, Mr, K, N, G, dtype, largest):
    g = torch.Generator(device="cuda").manual_seed(Mr + K)
    q = torch.randint(-128, 128, (Mr, K), dtype=torch.int8, device="cuda", generator=g)
    dy = torch.randn((Mr, N), device="cuda", generator=g).to(dtype)
    dy[Mr // 2, N // 2] = largest                                                # 3e19: in one row of tiles alone
    a, b = 0.5 + torch.rand(G, device="cuda", generator=g), -torch.rand(G, device="cuda", generator=g)
    dt = {torch.float16: M.F16, torch.bfloat16: M.BF16, torch.float32: M.F32}[dtype]
    ws = torch.empty(M.workspace_bytes(M.OP_LINEAR_DW_Q, Mr, K, N, dt), dtype=torch.uint8, device="cuda")
    out = torch.full((N * K + 128,), 7.0, device="cuda")
    bias = torch.full((N + 2,), 7.0, device="cuda")
    dW, db = out[64:64 + N * K].view(N, K), bias[1:1 + N]
    M.mesa_linear_dw_q(q, Mr, K, G, a, b, dy, N, dW, db, ws)
    x_hat = (q.double() + 128) * (a.double() / 255).repeat_interleave(K // G) + b.double().repeat_interleave(K // G)
    ref, d = dy.double().t().contiguous() @ x_hat, dy.double()
    # per row of dW, which shares its values of dy, against the row's sum of magnitudes (a row's own result may cancel)
    assert ((dW - ref).abs().amax(1) <= TOL * (d.abs().t().contiguous() @ x_hat.abs()).amax(1)).all()
    assert ((db - d.sum(0)).abs() <= TOL * d.abs().sum(0)).all()
    assert torch.all(out[:64] == 7) and torch.all(out[64 + N * K:] == 7) and bias[0] == 7 and bias[-1] == 7
    again = dW.clone()
    M.mesa_linear_dw_q(q, Mr, K, G, a, b, dy, N, dW, None, ws)                   # without the bias gradient: the same bits
    assert torch.equal(dW, again)
