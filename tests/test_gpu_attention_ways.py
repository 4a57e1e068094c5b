"""The attention products with heads enough for the kernels that go by tiles and for those that keep a head whole: lengths on either side of a
tile, a chunk and a vector, rows that start anywhere, against the same products in binary64; nothing outside an output is written and
nothing outside an input reaches a result."""
import pytest
import torch

from tests.test_gpu_parity import _mid_of_frame
from tests.test_gpu_shape_sweep import framed, intact

pytestmark = pytest.mark.gpu
BOUND = {torch.float16: 2e-3, torch.bfloat16: 1.6e-2}     # one rounding to the storage type and sums in binary32, as in the other parity tests


@pytest.fixture(scope="module")
def M():
    import paper_2111_11124_amd as m
    assert torch.cuda.is_available(), "these tests need the MI355X"
    m.lib()
    return m


def hat(q, a, b):
    return (q.double() + 128) * (a.double() / 255).view(1, -1, 1, 1) + b.double().view(1, -1, 1, 1)


def bmm(x, y):
    n = x.shape[0] * x.shape[1]
    return torch.bmm(x.reshape(n, *x.shape[2:]).contiguous(), y.reshape(n, *y.shape[2:]).contiguous()).view(*x.shape[:3], y.shape[3])


# heads: more than the 12288 to 28672 columns that the tiles ask for; 800 for the whole-head dQ; one image of many heads and many of few
@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16], ids=["f16", "bf16"])
@pytest.mark.parametrize("B,H,N,Dh", [(160, 3, 64, 64), (107, 3, 65, 96), (100, 3, 71, 128), (450, 1, 64, 32), (133, 6, 49, 64), (270, 3, 101, 64), (80, 3, 127, 32),
                                      (80, 3, 128, 64), (75, 3, 129, 64), (41, 5, 143, 96), (35, 4, 209, 128), (267, 3, 197, 64), (40, 3, 255, 64), (28, 4, 256, 64),
                                      (28, 4, 257, 64), (33, 2, 319, 32), (20, 3, 383, 96), (14, 3, 511, 128), (10, 5, 577, 64), (12, 4, 600, 64), (8, 4, 705, 96),
                                      (4, 7, 1031, 32), (5, 6, 1000, 64), (2, 13, 1001, 128)])
def test_attention_products_with_many_heads(M, B, H, N, Dh, dtype):
    g = torch.Generator(device="cuda").manual_seed(N * 1000 + Dh)
    aq = _mid_of_frame(torch.randint(-128, 128, (B, H, N, N), dtype=torch.int8, device="cuda", generator=g), 127)
    qq, kq, vq = (_mid_of_frame(torch.randint(-128, 128, (B, H, N, Dh), dtype=torch.int8, device="cuda", generator=g), 127) for _ in range(3))
    dO = _mid_of_frame(torch.randn((B, H, N, Dh), device="cuda", generator=g).to(dtype), float("nan"))
    dS = _mid_of_frame((torch.randn((B, H, N, N), device="cuda", generator=g) * 0.1).to(dtype), float("nan"))
    par = {k: (torch.linspace(1.0, 4.0, H, device="cuda") * s, torch.linspace(-2.0, -0.5, H, device="cuda") * s)
           for k, s in (("a", 0.25), ("q", 1.0), ("k", 1.5), ("v", 0.75))}
    outs = [framed(s, dtype) for s in ((B, H, N, N), (B, H, N, Dh), (B, H, N, Dh), (B, H, N, Dh))]
    dA, dV, dQ, dK = (o[1] for o in outs)
    M.mesa_attn_av_bwd_q(aq, vq, B, H, N, Dh, *par["a"], *par["v"], dO, dA, dV)
    M.mesa_attn_qk_bwd_q(qq, kq, B, H, N, Dh, *par["q"], *par["k"], dS, 0.2, dQ, dK)
    T = lambda t: t.transpose(2, 3)  # noqa: E731
    want = [lambda: bmm(dO.double(), T(hat(vq, *par["v"]))), lambda: bmm(T(hat(aq, *par["a"])), dO.double()), lambda: 0.2 * bmm(dS.double(), hat(kq, *par["k"])),
            lambda: 0.2 * bmm(T(dS.double()), hat(qq, *par["q"]))]
    for name, got, ref, (frame_, _) in zip(("dA", "dV", "dQ", "dK"), (dA, dV, dQ, dK), want, outs):
        r = ref()
        err = float((got.double() - r).abs().max() / r.abs().max())
        assert err <= BOUND[dtype], (name, err)
        assert intact(frame_), name
        del r


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16], ids=["f16", "bf16"])
def test_attention_products_with_a_map_larger_than_the_memory_side_cache(M, dtype):
    """dV before dA."""
    test_attention_products_with_many_heads(M, 1, 33, 2049, 32, dtype)
