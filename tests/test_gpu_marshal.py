"""The binding's native marshalling against its general path: the same results for every form both take, and what the native one
does not take raises what the general path raises."""
import ctypes

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def M():
    import paper_2111_11124_amd as m
    assert torch.cuda.is_available(), "these tests need the MI355X"
    m.lib()
    return m


class _Nothing:
    """leaves every call to the general path"""

    def __getattr__(self, name):
        return lambda *a: None


def _sequence(M, dtype, as_list):
    """every natively marshalled call once; the tensors they write"""
    g = torch.Generator(device="cuda").manual_seed(1)
    B, H, N, Dh, G = 2, 2, 24, 16, 2
    M_, D = B * N, H * Dh
    lay = [B, H, N * N] if as_list else (B, H, N * N)
    tok = (M_, G, D // G)
    x = torch.randn((B, H, N, N), device="cuda", generator=g).to(dtype)
    t = torch.randn((M_, D), device="cuda", generator=g).to(dtype)
    a, b, m = (torch.full((G,), v, device="cuda") for v in (6.0, -3.0, 3.0))
    ws = torch.empty(1 << 20, dtype=torch.uint8, device="cuda")
    q, q4 = torch.empty(x.numel(), dtype=torch.int8, device="cuda"), torch.empty(x.numel() // 2, dtype=torch.uint8, device="cuda")
    tq = torch.empty(t.numel(), dtype=torch.int8, device="cuda")
    out = [a, b, m]

    def new(like, dt=None, fill=0):
        o = torch.full_like(like, fill, dtype=dt)
        out.append(o)
        return o

    M.mesa_update_running_params(x, lay, a, b, 0.9, True, ws)
    M.mesa_update_running_params(x, lay, a, b, 1, 0, ws)
    M.mesa_update_running_params_sym(x, lay, a, b, 0.5, False, ws)
    M.mesa_update_running_params_fixed_beta(x, lay, a, b, 0.5, False, -3, ws)
    M.mesa_update_running_params_static(x, lay, a, b, 0.5, False)
    M.mesa_update_running_scale_sym(x, lay, m, 0.5, False, ws)
    M.mesa_quantize_headwise(x, lay, a, b, q, M.ROUND_STOCHASTIC, 1 << 63, 7)
    M.mesa_quantize_headwise(x, lay, a, b, new(q), seed=-5)
    M.mesa_quantize_headwise_b4(x, lay, a, b, q4)
    M.mesa_quantize_sym(x, lay, m, new(q))
    M.mesa_quantize_update_fused(t, tok, a, b, 0.9, tq, ws, offset=3)
    M.mesa_dequantize(q, lay, a, b, new(x))
    M.mesa_dequantize_b4(q4, lay, a, b, new(x))
    M.mesa_dequantize_sym(q, lay, m, new(x))
    M.mesa_gelu_fwd_q(t, tok, a, b, 0.9, new(t), new(tq), ws)
    M.mesa_softmax_fwd_q(x, B, H, N, N, a, b, 0.9, new(x), new(q), ws)
    gamma = torch.ones(D, device="cuda").to(dtype)
    mean, rstd = torch.zeros(M_, device="cuda"), torch.ones(M_, device="cuda")
    M.mesa_layernorm_fwd_q(t, M_, D, G, gamma, gamma, 1e-5, a, b, 0.9, new(t), new(mean), new(mean), new(tq), ws)
    M.mesa_gelu_bwd_q(tq, tok, a, b, t, new(t))
    M.mesa_gelu_bwd_q_b4(q4, lay, a, b, x, new(x))
    M.mesa_relu_bwd_q(tq, tok, a, b, t, new(t))
    M.mesa_softmax_bwd_q(q, B, H, N, N, a, b, x, new(x))
    M.mesa_layernorm_bwd_q(tq, M_, D, G, a, b, mean, rstd, gamma, t, new(t), new(gamma, torch.float32), new(gamma, torch.float32), ws)
    for bias in (torch.empty(D, device="cuda"), None):
        M.mesa_linear_dw_q(tq, M_, D, G, a, b, t, D, new(torch.empty(D, D, device="cuda")), bias, ws)
        out += [] if bias is None else [bias]
    cv = M.Conv2d(B, 4, 8, 8, 4, 3, 3, 1, 1, 1, 1, 1, 1)
    M.mesa_conv2d_dw_q(q[:B * 4 * 64], cv, 2, a, b, x.view(-1)[:B * 4 * 64], new(torch.empty(4, 4, 3, 3, device="cuda")), None, ws)
    hq = tq.view(-1)
    M.mesa_attn_av_bwd_q(q, hq, B, H, N, Dh, a, b, a, b, t, new(x), new(t))
    M.mesa_attn_qk_bwd_q(hq, hq, B, H, N, Dh, a, b, a, b, x, 0.25, new(t), new(t))
    torch.cuda.synchronize()
    return [o.float().cpu().numpy() for o in out + [q, q4, tq]]


@pytest.mark.parametrize("dtype", [torch.float32, torch.float16, torch.bfloat16], ids=["f32", "f16", "bf16"])
def test_native_and_general_marshalling_make_the_same_calls(M, dtype, monkeypatch):
    from paper_2111_11124_amd import _ffi
    native = _sequence(M, dtype, False)
    with torch.cuda.stream(torch.cuda.Stream()):       # a stream of its own
        other = _sequence(M, dtype, True)
    monkeypatch.setattr(_ffi, "_fast", _Nothing())
    general = _sequence(M, dtype, False)
    for u, v, w in zip(native, other, general):
        assert np.array_equal(u, v, equal_nan=True) and np.array_equal(u, w, equal_nan=True)


def test_what_the_native_marshalling_does_not_take(M):
    x = torch.zeros((4, 64), device="cuda")
    a, q = torch.ones(1, device="cuda"), torch.zeros(256, dtype=torch.int8, device="cuda")
    lay = (4, 1, 64)
    M.mesa_quantize_headwise(x, np.array(lay).tolist(), a, a, q)
    with pytest.raises(ValueError, match="device tensors"):
        M.mesa_quantize_headwise(x.cpu(), lay, a, a, q)
    with pytest.raises(ValueError, match="contiguous"):
        M.mesa_quantize_headwise(x.t(), lay, a, a, q)
    with pytest.raises(TypeError, match="unsupported dtype"):
        M.mesa_quantize_headwise(x.double(), lay, a, a, q)
    with pytest.raises(TypeError):
        M.mesa_quantize_headwise(x, (4, 1, 64.0), a, a, q)
    with pytest.raises(TypeError):
        M.mesa_quantize_headwise(x, (4, 1, 64, 1), a, a, q)
    with pytest.raises(ctypes.ArgumentError):
        M.mesa_softmax_bwd_q(q, 1, 1, 4, 64.0, a, a, x, x)
    with pytest.raises(AssertionError):
        M.mesa_gelu_bwd_q(q, lay, a, a, x, x.half())
    for bad in (None, a.view(torch.int8)[1:2]):        # null, misaligned: the library's own answer
        with pytest.raises(M.MesaError) as e:
            M.mesa_quantize_headwise(x, lay, bad, a, q)
        assert e.value.status == M.ERR_INVALID_ARG
