"""Attention products of equal heads: a head's result does not depend on where in the batch it stands.  Every kernel sums in an order of its own, but the same
one for every head, so the results are the same bits.  Row tiles per head (64 rows) that are and are no multiple of 16, with whole chunks of columns and without."""
import pytest
import torch

from tests.test_gpu_parity import M  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16], ids=["f16", "bf16"])
@pytest.mark.parametrize("B,H,N,Dh", [(40, 4, 197, 64), (30, 4, 320, 64), (24, 3, 576, 32), (10, 4, 1024, 64), (8, 4, 1088, 64), (6, 3, 2048, 64), (2, 3, 3072, 32), (4, 3, 2112, 96),
                                      (2, 3, 4096, 128)])
def test_equal_heads_give_equal_results(M, B, H, N, Dh, dtype):  # noqa: F811
    g = torch.Generator(device="cuda").manual_seed(N + Dh)
    one = lambda *s: torch.randint(-128, 128, s, dtype=torch.int8, device="cuda", generator=g)  # noqa: E731
    heads = lambda t: t.expand(B, H, *t.shape[-2:]).contiguous()  # noqa: E731
    a, q, k, v = (heads(t) for t in (one(N, N), one(N, Dh), one(N, Dh), one(N, Dh)))
    s, o = torch.full((H,), 0.7, device="cuda"), torch.full((H,), -0.3, device="cuda")
    dO, dS = (heads(torch.randn(N, n, device="cuda", generator=g).to(dtype)) for n in (Dh, N))
    dA, dV, dQ, dK = torch.empty_like(dS), torch.empty_like(dO), torch.empty_like(dO), torch.empty_like(dO)
    M.mesa_attn_av_bwd_q(a, v, B, H, N, Dh, s, o, s, o, dO, dA, dV)
    M.mesa_attn_qk_bwd_q(q, k, B, H, N, Dh, s, o, s, o, dS, Dh ** -0.5, dQ, dK)
    for name, t in dict(dA=dA, dV=dV, dQ=dQ, dK=dK).items():
        assert torch.equal(t, t[:1, :1].expand_as(t)), name
