"""The attention products of few heads, a 32 x 32 tile per workgroup of four, eight or sixteen waves that share out the contraction: blocks of
16 steps that end inside, at and behind the extents, rows that start anywhere, both sides of the lines to the other kernels, values of
binary32 that are too large to be cut; against the same products in binary64, and nothing outside an output is written and nothing
outside an input reaches a result."""
import pytest
import torch

from tests.test_gpu_attention_ways import bmm, hat
from tests.test_gpu_parity import _mid_of_frame
from tests.test_gpu_shape_sweep import framed, intact

pytestmark = pytest.mark.gpu
# one rounding to the storage type and sums in binary32, as in the other parity tests
BOUND = {torch.float16: 2e-3, torch.bfloat16: 1.6e-2, torch.float32: 1e-5}


@pytest.fixture(scope="module")
def M():
    import paper_2111_11124_amd as m
    assert torch.cuda.is_available(), "these tests need the MI355X"
    m.lib()
    return m


def run(M, B, H, N, Dh, dtype, large):
    g = torch.Generator(device="cuda").manual_seed(N * 1000 + Dh)
    aq = _mid_of_frame(torch.randint(-128, 128, (B, H, N, N), dtype=torch.int8, device="cuda", generator=g), 127)
    qq, kq, vq = (_mid_of_frame(torch.randint(-128, 128, (B, H, N, Dh), dtype=torch.int8, device="cuda", generator=g), 127) for _ in range(3))
    dO, dS = torch.randn((B, H, N, Dh), device="cuda", generator=g).to(dtype), (torch.randn((B, H, N, N), device="cuda", generator=g) * 0.1).to(dtype)
    if large:
        dO[0, 0, N // 2, Dh // 2] = dS[-1, -1, N - 1, N // 3] = 3e19
    dO, dS = _mid_of_frame(dO, float("nan")), _mid_of_frame(dS, float("nan"))
    par = {k: (torch.linspace(1.0, 4.0, H, device="cuda") * s, torch.linspace(-2.0, -0.5, H, device="cuda") * s)
           for k, s in (("a", 0.25), ("q", 1.0), ("k", 1.5), ("v", 0.75))}
    outs = [framed(s, dtype) for s in ((B, H, N, N), (B, H, N, Dh), (B, H, N, Dh), (B, H, N, Dh))]
    dA, dV, dQ, dK = (o[1] for o in outs)
    M.mesa_attn_av_bwd_q(aq, vq, B, H, N, Dh, *par["a"], *par["v"], dO, dA, dV)
    M.mesa_attn_qk_bwd_q(qq, kq, B, H, N, Dh, *par["q"], *par["k"], dS, 0.2, dQ, dK)
    T = lambda t: t.transpose(2, 3)  # noqa: E731
    d, ds = dO.double(), dS.double()
    terms = [(d, T(hat(vq, *par["v"])), 1.0), (T(hat(aq, *par["a"])), d, 1.0), (ds, hat(kq, *par["k"]), 0.2), (T(ds), hat(qq, *par["q"]), 0.2)]
    for name, got, (x, y, f), (frame_, _) in zip(("dA", "dV", "dQ", "dK"), (dA, dV, dQ, dK), terms, outs):
        ref, got = f * bmm(x, y), got.double()
        # a large value is in one row of dA, dQ and dK and in one column of dV: the others are to be right for themselves
        along = 3 if name != "dV" else 2
        size = (f * bmm(x.abs(), y.abs())).amax(along) if large else ref.abs().max()
        assert ((got - ref).abs().amax(along) <= BOUND[dtype] * size).all(), name
        assert intact(frame_), name


@pytest.mark.parametrize("dtype,large", [(torch.float16, False), (torch.bfloat16, False), (torch.float32, False), (torch.float32, True)],
                         ids=["f16", "bf16", "f32", "f32 large"])
@pytest.mark.parametrize("B,H,N,Dh", [
    (1, 1, 8, 8), (1, 3, 15, 24), (2, 1, 17, 64), (1, 2, 31, 65), (3, 1, 33, 33), (1, 2, 64, 96), (2, 2, 65, 64), (1, 1, 127, 128), (1, 2, 128, 130), (1, 3, 129, 40),
    (2, 3, 197, 64), (1, 1, 257, 64), (1, 2, 513, 32), (1, 1, 1031, 64),
    (16, 4, 128, 64), (13, 5, 127, 64), (16, 2, 256, 64), (16, 1, 256, 64), (17, 1, 255, 64),       # 512 and 256 tiles, and more
    (10, 10, 128, 64), (21, 5, 120, 64), (8, 4, 250, 64), (9, 12, 197, 64),                          # 800 and more; beyond them all
    (53, 4, 64, 32), (17, 3, 128, 64), (9, 4, 150, 32)])
def test_attention_products_with_few_heads(M, B, H, N, Dh, dtype, large):
    run(M, B, H, N, Dh, dtype, large)
