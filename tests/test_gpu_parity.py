"""GPU parity: libmesa (through its C ABI) against the CPU oracle on the same seeded inputs.

Codes, running parameters and mesa_dequantize output must match bit for bit; gradients within
max|gpu - ref| / max|ref| <= 1e-5 (binary32 storage), 2e-3 (binary16 storage) or 1.6e-2 (bfloat16
storage: four roundings of 2^-8, as 2e-3 is four of 2^-11).  numpy has no bfloat16: the oracle is given
the stored values widened to binary32, which is exact, so codes and parameters are still bit for bit.
"""
import numpy as np
import pytest
import torch

import mesa_workloads as W
from oracle import mesa_ref as R

pytestmark = pytest.mark.gpu

TOL = {torch.float32: 1e-5, torch.float16: 2e-3, torch.bfloat16: 1.6e-2}
DTYPES = [torch.float32, torch.float16, torch.bfloat16]
DTYPE_IDS = ["f32", "f16", "bf16"]


def npy(t):
    """A tensor's values as a numpy array; bfloat16 widened to binary32 (exact)."""
    return (t.float() if t.dtype == torch.bfloat16 else t).cpu().numpy()


@pytest.fixture(scope="module")
def M():
    import paper_2111_11124_amd as m
    assert torch.cuda.is_available(), "these tests need the MI355X"
    m.lib()
    return m


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def canon(a):
    """-0.0 -> +0.0 (the library returns a minimum of -0.0 as +0.0)."""
    return (np.asarray(a, np.float32) + np.float32(0.0)).view(np.uint32)


def relerr(got, ref):
    got = np.asarray(got, np.float64)
    return float(np.abs(got - ref).max() / max(np.abs(ref).max(), 1e-30))


def ws_for(m, op, d0, d1, d2, dt=None):
    n = m.workspace_bytes(op, d0, d1, d2, {None: m.F16, torch.float16: m.F16, torch.bfloat16: m.BF16, torch.float32: m.F32}[dt])
    return torch.empty(max(n, 16), dtype=torch.uint8, device="cuda")


def run_params(m, xs, layout, lam=0.9):
    """first_call update on xs[0], EMA updates on the rest; returns (gpu alpha, beta) and the oracle's."""
    G = layout[1]
    a = torch.full((G,), 123.0, device="cuda")
    b = torch.full((G,), -77.0, device="cuda")
    ra, rb = np.full(G, 123.0, np.float32), np.full(G, -77.0, np.float32)
    ws = ws_for(m, m.OP_UPDATE_RUNNING_PARAMS, *layout)
    for i, x in enumerate(xs):
        m.mesa_update_running_params(x, layout, a, b, lam, i == 0, ws)
        ra, rb = R.update_running_params(npy(x), layout, ra, rb, lam, i == 0)
    torch.cuda.synchronize()
    return a, b, ra, rb


LAYOUTS = [
    (3, 4, 1000),      # slabs of whole vectors
    (5, 3, 361),       # odd slabs: vectors straddle heads (19 x 19 attention)
    (37, 6, 64),       # channel groups of a (37, 384) token matrix
    (50, 3, 32),
    (1, 1, 12345),     # one group, ragged tail
    (7, 5, 3),         # slabs shorter than a vector
    (2, 2, 70001),
    (3000, 12, 256),   # several grid steps
]


@pytest.mark.parametrize("dtype", DTYPES, ids=DTYPE_IDS)
@pytest.mark.parametrize("layout", LAYOUTS)
def test_params_codes_and_dequantize_are_bit_exact(M, layout, dtype):
    outer, G, inner = layout
    n = outer * G * inner
    g = torch.Generator(device="cuda").manual_seed(n)
    scale = torch.tensor([0.3, 1.0, 4.0, 11.0, 0.05, 2.0, 7.0, 1.5, 0.8, 3.0, 0.1, 6.0], device="cuda")[:G].view(1, G, 1)
    xs = [(torch.randn((outer, G, inner), generator=g, device="cuda") * scale + 0.25 * i).to(dtype).contiguous()
          for i in range(3)]
    a, b, ra, rb = run_params(M, xs, layout)
    assert np.array_equal(canon(npy(a)), canon(ra)), (npy(a), ra)
    assert np.array_equal(canon(npy(b)), canon(rb)), (npy(b), rb)

    x = xs[-1]
    xh = npy(x)
    an, bn = npy(a), npy(b)
    for mode, seed, off in ((M.ROUND_NEAREST_EVEN, 0, 0), (M.ROUND_STOCHASTIC, 0xDEADBEEF12345, (1 << 33) + 17)):
        q = torch.empty(n, dtype=torch.int8, device="cuda")
        M.mesa_quantize_headwise(x, layout, a, b, q, mode, seed, off)
        rq = R.quantize_headwise(xh, layout, an, bn, mode, seed, off).reshape(-1)
        got = npy(q)
        bad = np.nonzero(got != rq)[0]
        assert bad.size == 0, (mode, bad[:10], got[bad[:10]], rq[bad[:10]])
    for odt in (torch.float32, torch.float16):
        out = torch.empty(n, dtype=odt, device="cuda")
        M.mesa_dequantize(q, layout, a, b, out)
        ref = R.dequantize(rq, layout, an, bn, np.float32 if odt == torch.float32 else np.float16)
        u = np.uint32 if odt == torch.float32 else np.uint16
        assert np.array_equal(npy(out).view(u), ref.view(u))
    out = torch.empty(n, dtype=torch.bfloat16, device="cuda")
    M.mesa_dequantize(q, layout, a, b, out)
    assert np.array_equal(out.view(torch.int16).cpu().numpy().view(np.uint16), R.dequantize(rq, layout, an, bn, "bf16").reshape(-1))


def block_parity(m, spec, modes=("nearest", "stochastic")):
    """The whole path on one block's saved-activation set, every output against the oracle."""
    dt = spec.dtype
    tol = TOL[dt]
    H = spec.heads
    report = {}

    def params_and_codes(draws, layout, mode, seed, off):
        a, b, ra, rb = run_params(m, draws, layout, spec.lam)
        assert np.array_equal(canon(npy(a)), canon(ra)) and np.array_equal(canon(npy(b)), canon(rb))
        x = draws[-1]
        q = torch.empty(x.numel(), dtype=torch.int8, device="cuda")
        m.mesa_quantize_headwise(x, layout, a, b, q, mode, seed, off)
        rq = R.quantize_headwise(npy(x), layout, ra, rb, mode, seed, off).reshape(-1)
        assert np.array_equal(npy(q), rq)
        return a, b, ra, rb, q, rq

    for mi, mode_name in enumerate(modes):
        mode = m.ROUND_NEAREST_EVEN if mode_name == "nearest" else m.ROUND_STOCHASTIC
        seed = 1000 + spec.seed
        # --- attention map -> softmax backward
        B, Hh, rows, cols = spec.attn
        draws = [W.attention_map(spec, d, "cuda") for d in range(3)]
        a, b, ra, rb, q, rq = params_and_codes(draws, spec.attn_layout, mode, seed, 0)
        assert (npy(b) >= 0).all()
        del draws
        dy = W.upstream_grad(spec, "dy_attn", spec.attn, "cuda")
        dx = torch.empty_like(dy)
        m.mesa_softmax_bwd_q(q, B, Hh, rows, cols, a, b, dy, dx)
        ref = R.softmax_bwd_q(rq, B, Hh, rows, cols, ra, rb, npy(dy))
        report[f"softmax_{mode_name}"] = relerr(npy(dx).reshape(ref.shape), ref)
        del dy, dx, ref
        # --- GELU input -> GELU backward
        lay = spec.gelu_layout
        draws = [W.gelu_input(spec, d, "cuda") for d in range(3)]
        a, b, ra, rb, q, rq = params_and_codes(draws, lay, mode, seed, 1 << 40)
        del draws
        dy = W.upstream_grad(spec, "dy_gelu", (spec.tokens, spec.mlp), "cuda")
        dx = torch.empty_like(dy)
        m.mesa_gelu_bwd_q(q, lay, a, b, dy, dx)
        ref = R.gelu_bwd_q(rq, lay, ra, rb, npy(dy))
        report[f"gelu_{mode_name}"] = relerr(npy(dx).reshape(ref.shape), ref)
        del dy, dx, ref
        # --- LayerNorm input -> LayerNorm backward
        lay = spec.ln_layout
        Mr, D = spec.tokens, spec.dim
        draws = [W.token_matrix(spec, "ln", d, "cuda") for d in range(3)]
        a, b, ra, rb, q, rq = params_and_codes(draws, lay, mode, seed, 2 << 40)
        mean, rstd = W.layernorm_stats(draws[-1])
        del draws
        gamma = W.layernorm_gamma(spec, "cuda")
        dy = W.upstream_grad(spec, "dy_ln", (Mr, D), "cuda")
        dx = torch.empty_like(dy)
        dg = torch.empty(D, device="cuda")
        db = torch.empty(D, device="cuda")
        ws = ws_for(m, m.OP_LAYERNORM_BWD_Q, Mr, D, H)
        m.mesa_layernorm_bwd_q(q, Mr, D, H, a, b, mean, rstd, gamma, dy, dx, dg, db, ws)
        rdx, rdg, rdb = R.layernorm_bwd_q(rq, Mr, D, H, ra, rb, npy(mean), npy(rstd),
                                          npy(gamma), npy(dy))
        report[f"ln_dx_{mode_name}"] = relerr(npy(dx), rdx)
        report[f"ln_dgamma_{mode_name}"] = relerr(npy(dg), rdg)
        report[f"ln_dbeta_{mode_name}"] = relerr(npy(db), rdb)
        del dy, dx
        # --- Linear inputs -> dW (entries sampled when the full matrix is out of the oracle's reach)
        for li, (K, N) in enumerate(spec.linears):
            lay = (Mr, H, K // H)
            draws = [W.token_matrix(spec, "lin", 10 * li + d, "cuda", width=K) for d in range(3)]
            a, b, ra, rb, q, rq = params_and_codes(draws, lay, mode, seed, (3 + li) << 40)
            del draws
            dy = W.upstream_grad(spec, "dy_lin", (Mr, N), "cuda")
            dW = torch.empty((N, K), device="cuda")
            dbias = torch.empty(N, device="cuda")
            ws = ws_for(m, m.OP_LINEAR_DW_Q, Mr, K, N, dt)
            m.mesa_linear_dw_q(q, Mr, K, H, a, b, dy, N, dW, dbias, ws)
            dyh = npy(dy)
            got = npy(dW).astype(np.float64)
            if Mr * K * N <= 4e9:
                rW, rb_ = R.linear_dw_q(rq, Mr, K, H, ra, rb, dyh, N)
                report[f"dw{li}_{mode_name}"] = relerr(got, rW)
            else:
                rng = np.random.default_rng(li)
                n_idx = np.concatenate([np.repeat(rng.integers(0, N, 4), K), rng.integers(0, N, 4096)])
                k_idx = np.concatenate([np.tile(np.arange(K), 4), rng.integers(0, K, 4096)])
                ent = R.linear_dw_q_entries(rq, Mr, K, H, ra, rb, dyh, N, n_idx, k_idx)
                scale = max(np.abs(ent).max(), 1e-30)
                report[f"dw{li}_{mode_name}"] = float(np.abs(got[n_idx, k_idx] - ent).max() / scale)
                rb_ = dyh.astype(np.float64).sum(0)
            report[f"db{li}_{mode_name}"] = relerr(npy(dbias), rb_)
            del dy, dW
        if mi == 0:
            # mesa_dequantize on the last codes, both output types, bit for bit
            for odt, npo, u in ((torch.float32, np.float32, np.uint32), (torch.float16, np.float16, np.uint16)):
                out = torch.empty(q.numel(), dtype=odt, device="cuda")
                m.mesa_dequantize(q, lay, a, b, out)
                assert np.array_equal(npy(out).view(u), R.dequantize(rq, lay, ra, rb, npo).view(u))
            out = torch.empty(q.numel(), dtype=torch.bfloat16, device="cuda")
            m.mesa_dequantize(q, lay, a, b, out)
            assert np.array_equal(out.view(torch.int16).cpu().numpy().view(np.uint16), R.dequantize(rq, lay, ra, rb, "bf16").reshape(-1))
    bad = {k: v for k, v in report.items() if not v <= tol}
    assert not bad, (bad, report)
    return report


def test_config1_deit_ti_block_fp32(M):
    print(block_parity(M, W.CONFIGS[1]))


def test_tiny_ragged_block_every_dtype(M):
    for dt in DTYPES:
        print(block_parity(M, W.small_case(dt, B=3, H=3, N=19, D=48, mlp=96)))


def test_config2_deit_s_shape_batch8(M):
    print(block_parity(M, W.scaled(W.CONFIGS[2], 16)))


def test_config2_deit_s_shape_batch8_bfloat16(M):
    from dataclasses import replace
    print(block_parity(M, replace(W.scaled(W.CONFIGS[2], 16), dtype=torch.bfloat16), modes=("stochastic",)))


def test_config3_swin_t_shape_reduced(M):
    print(block_parity(M, W.scaled(W.CONFIGS[3], 64), modes=("stochastic",)))


def test_config4_deit_b_shape_batch4(M):
    print(block_parity(M, W.scaled(W.CONFIGS[4], 64), modes=("stochastic",)))


def test_config5_long_sequence_shape_reduced(M):
    spec = W.scaled(W.CONFIGS[5], 8)       # one sample: attention map (1, 16, 4096, 4096)
    from dataclasses import replace
    spec = replace(spec, attn=(1, 16, 512, 4096))   # 512 of the 4096 query rows per head
    print(block_parity(M, spec, modes=("stochastic",)))


def _ln_case(M, spec, G):
    """LayerNorm backward alone on one token matrix: dx, dgamma, dbeta against the oracle."""
    Mr, D = spec.tokens, spec.dim
    lay = (Mr, G, D // G)
    draws = [W.token_matrix(spec, "ln", d, "cuda") for d in range(2)]
    a, b, ra, rb = run_params(M, draws, lay, spec.lam)
    x = draws[-1]
    q = torch.empty(x.numel(), dtype=torch.int8, device="cuda")
    M.mesa_quantize_headwise(x, lay, a, b, q, M.ROUND_STOCHASTIC, 5, 0)
    rq = npy(q)
    mean, rstd = W.layernorm_stats(x)
    gamma = W.layernorm_gamma(spec, "cuda")
    dy = W.upstream_grad(spec, "dy_ln", (Mr, D), "cuda")
    dx = torch.empty_like(dy)
    dg = torch.empty(D, device="cuda")
    db = torch.empty(D, device="cuda")
    ws = ws_for(M, M.OP_LAYERNORM_BWD_Q, Mr, D, G)
    M.mesa_layernorm_bwd_q(q, Mr, D, G, a, b, mean, rstd, gamma, dy, dx, dg, db, ws)
    rdx, rdg, rdb = R.layernorm_bwd_q(rq, Mr, D, G, ra, rb, npy(mean), npy(rstd),
                                      npy(gamma), npy(dy))
    return {"dx": relerr(npy(dx), rdx), "dgamma": relerr(npy(dg), rdg), "dbeta": relerr(npy(db), rdb)}


@pytest.mark.parametrize("dtype", DTYPES, ids=DTYPE_IDS)
@pytest.mark.parametrize("D,G,tokens", [(8, 1, 37), (48, 3, 57), (128, 4, 333), (192, 3, 1000), (384, 6, 1579), (512, 8, 130),
                                        (768, 12, 517), (1024, 16, 259), (1032, 3, 77), (2048, 16, 35), (4096, 8, 19)])
def test_layernorm_bwd_every_row_length_class(M, D, G, tokens, dtype):
    """Rows of 1..128 vectors go through lane groups of 8, 16, 32 or 64 lanes (one or two vectors per lane),
    longer rows through workgroup tiles; ragged row counts in every class."""
    spec = W.small_case(dtype, seed=D + tokens, B=1, H=G, N=tokens, D=D, mlp=D)
    rep = _ln_case(M, spec, G)
    assert all(v <= TOL[dtype] for v in rep.values()), rep


@pytest.mark.parametrize("dtype", DTYPES, ids=DTYPE_IDS)
@pytest.mark.parametrize("D,G,tokens", [(100, 5, 37), (7, 1, 5), (120, 3, 1030), (4104, 3, 9), (8192, 16, 6), (5000, 8, 11)])
def test_layernorm_bwd_rows_the_vector_kernels_cannot_take(M, D, G, tokens, dtype):
    """Row lengths and group widths that are no multiple of 8, rows above 4096 elements: the plain kernels."""
    spec = W.small_case(dtype, seed=D + tokens, B=1, H=G, N=tokens, D=D, mlp=D)
    rep = _ln_case(M, spec, G)
    assert all(v <= TOL[dtype] for v in rep.values()), rep


@pytest.mark.parametrize("Mr,K,N", [(31, 16, 8), (32, 48, 24), (97, 128, 264), (100 * 32, 384, 256), (101 * 32 + 5, 256, 520),
                                    (4 * 32 * 7 + 13, 784, 136), (9000, 272, 1000)])
@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16], ids=["f16", "bf16"])
def test_linear_dw_ragged_shapes(M, Mr, K, N, dtype):
    """Slices of 1, 2 and 3k stages, a ragged last stage, K and N that leave partial tiles; both 16-bit types.
    The products are exact and the sums binary32 for either type, so both meet the binary16 bound."""
    H = 1 if K % 3 else 3
    spec = W.small_case(dtype, seed=Mr + K, B=1, H=H, N=Mr, D=K, mlp=N)
    lay = (Mr, H, K // H)
    draws = [W.token_matrix(spec, "lin", d, "cuda", width=K) for d in range(2)]
    a, b, ra, rb = run_params(M, draws, lay, spec.lam)
    q = torch.empty(Mr * K, dtype=torch.int8, device="cuda")
    M.mesa_quantize_headwise(draws[-1], lay, a, b, q, M.ROUND_STOCHASTIC, 9, 0)
    rq = npy(q)
    dy = W.upstream_grad(spec, "dy_lin", (Mr, N), "cuda")
    dW = torch.empty((N, K), device="cuda")
    dbias = torch.empty(N, device="cuda")
    ws = ws_for(M, M.OP_LINEAR_DW_Q, Mr, K, N, dtype)
    M.mesa_linear_dw_q(q, Mr, K, H, a, b, dy, N, dW, dbias, ws)
    rW, rb_ = R.linear_dw_q(rq, Mr, K, H, ra, rb, npy(dy), N)
    rep = {"dW": relerr(npy(dW).astype(np.float64), rW), "db": relerr(npy(dbias), rb_)}
    assert all(v <= TOL[torch.float16] for v in rep.values()), rep


@pytest.mark.parametrize("dtype", DTYPES, ids=DTYPE_IDS)
@pytest.mark.parametrize("layout", [(3, 3, 19 * 19), (57, 3, 32), (5, 7, 1000), (1, 4, 8), (2, 6, 197 * 197), (1579, 6, 64)])
def test_single_pass_forward_matches_the_oracle_bit_for_bit(M, layout, dtype):
    """mesa_quantize_update_fused: codes with the parameters on entry and the moved parameters, three steps
    in a row, both rounding modes; and the same codes / parameters as the two calls it combines."""
    n = layout[0] * layout[1] * layout[2]
    g = torch.Generator(device="cuda").manual_seed(n)
    xs = [(torch.randn(n, generator=g, device="cuda") * (1 + t)).to(dtype) for t in range(4)]
    a, b, ra, rb = run_params(M, xs[:1], layout)          # first call: the two-call order
    ws = ws_for(M, M.OP_UPDATE_RUNNING_PARAMS, *layout)
    for t in range(1, 4):
        mode = M.ROUND_STOCHASTIC if t % 2 else M.ROUND_NEAREST_EVEN
        q2 = torch.empty(n, dtype=torch.int8, device="cuda")
        M.mesa_quantize_headwise(xs[t], layout, a, b, q2, mode, 77, 1000 * t)     # the two calls, for comparison
        a2, b2 = a.clone(), b.clone()
        M.mesa_update_running_params(xs[t], layout, a2, b2, 0.9, False, ws)
        q = torch.empty(n, dtype=torch.int8, device="cuda")
        M.mesa_quantize_update_fused(xs[t], layout, a, b, 0.9, q, ws, mode, 77, 1000 * t)
        rq, ra, rb = R.quantize_update_fused(npy(xs[t]), layout, ra, rb, 0.9, mode, 77, 1000 * t)
        assert np.array_equal(npy(q), rq.reshape(-1))
        assert np.array_equal(canon(npy(a)), canon(ra)) and np.array_equal(canon(npy(b)), canon(rb))
        assert torch.equal(q, q2) and torch.equal(a, a2) and torch.equal(b, b2)


@pytest.mark.parametrize("dtype", DTYPES, ids=DTYPE_IDS)
def test_per_sample_statistics_through_the_layout_descriptor(M, dtype):
    """One (alpha, beta) pair per sample and head -- the paper's per-sample ablation -- is the layout
    (1, B*H, inner): parameters, codes, softmax backward (B = 1, H = B*H) and GELU backward with more
    groups than its table holds (direct evaluation of the derivative)."""
    B, H, N = 16, 6, 19
    G = B * H
    lay = (1, G, N * N)
    gen = torch.Generator(device="cuda").manual_seed(5)
    logits = torch.randn((B, H, N, N), generator=gen, device="cuda") * torch.linspace(0.3, 5.0, G, device="cuda").view(B, H, 1, 1)
    xs = [torch.softmax(logits + 0.1 * t, dim=-1).to(dtype).contiguous() for t in range(2)]
    a, b, ra, rb = run_params(M, xs, lay)
    assert np.array_equal(canon(npy(a)), canon(ra)) and np.array_equal(canon(npy(b)), canon(rb))
    assert len(set(np.round(ra, 6))) > G // 2          # the samples really have their own ranges
    q = torch.empty(xs[-1].numel(), dtype=torch.int8, device="cuda")
    M.mesa_quantize_headwise(xs[-1], lay, a, b, q, M.ROUND_STOCHASTIC, 3, 0)
    rq = R.quantize_headwise(npy(xs[-1]), lay, ra, rb, R.ROUND_STOCHASTIC, 3, 0).reshape(-1)
    assert np.array_equal(npy(q), rq)
    dy = torch.randn((B, H, N, N), generator=gen, device="cuda").to(dtype)
    dx = torch.empty_like(dy)
    M.mesa_softmax_bwd_q(q, 1, G, N, N, a, b, dy, dx)
    ref = R.softmax_bwd_q(rq, 1, G, N, N, ra, rb, npy(dy))
    assert relerr(npy(dx).reshape(ref.shape), ref) <= TOL[dtype]
    # GELU input with 96 groups of 40 channels
    lay2 = (50, G, 40)
    x = (torch.randn(lay2, generator=gen, device="cuda") * 1.5).to(dtype).contiguous()
    a2, b2, ra2, rb2 = run_params(M, [x], lay2)
    q2 = torch.empty(x.numel(), dtype=torch.int8, device="cuda")
    M.mesa_quantize_headwise(x, lay2, a2, b2, q2, M.ROUND_NEAREST_EVEN, 0, 0)
    rq2 = R.quantize_headwise(npy(x), lay2, ra2, rb2, R.ROUND_NEAREST, 0, 0).reshape(-1)
    assert np.array_equal(npy(q2), rq2)
    dy2 = torch.randn(lay2, generator=gen, device="cuda").to(dtype)
    dx2 = torch.empty_like(dy2)
    M.mesa_gelu_bwd_q(q2, lay2, a2, b2, dy2, dx2)
    ref2 = R.gelu_bwd_q(rq2, lay2, ra2, rb2, npy(dy2))
    assert relerr(npy(dx2).reshape(ref2.shape), ref2) <= TOL[dtype]


@pytest.mark.parametrize("B,H,N,Dh", [(2, 3, 19, 8), (3, 6, 197, 64), (2, 4, 64, 32), (1, 2, 130, 100), (5, 3, 49, 32), (1, 2, 300, 128), (2, 2, 33, 48), (1, 3, 40, 96), (3, 2, 40, 64), (2, 2, 8, 32), (1, 1, 65, 32), (1, 2, 24, 128), (1, 1, 255, 128), (1, 2, 223, 32), (2, 1, 224, 64), (1, 1, 256, 96)])
def test_attention_matmul_backward_against_the_oracle(M, B, H, N, Dh):
    """dA, dV of O = A V and dQ, dK of S = scale Q K^T at head-wise codes (binary16), chained through the
    library's own softmax backward as a training step would."""
    _attention_case(M, B, H, N, Dh, torch.float16)


@pytest.mark.parametrize("B,H,N,Dh", [(2, 3, 19, 8), (2, 6, 197, 64), (3, 3, 49, 32), (1, 2, 130, 100), (1, 1, 65, 96), (1, 2, 8, 128),
                                      (2, 4, 64, 32), (1, 2, 300, 128), (3, 2, 40, 64), (1, 2, 24, 128), (1, 1, 255, 128), (1, 2, 223, 32),
                                      (2, 1, 224, 64), (1, 1, 256, 96)])
def test_attention_matmul_backward_bfloat16(M, B, H, N, Dh):
    """The same products on bfloat16 tensors."""
    _attention_case(M, B, H, N, Dh, torch.bfloat16)


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16], ids=["f16", "bf16"])
@pytest.mark.parametrize("B,H,N,Dh", [(1, 2, 272, 64), (1, 1, 512, 32), (1, 2, 528, 128), (1, 1, 1024, 64), (2, 1, 304, 64), (1, 3, 288, 32),
                                      (1, 1, 784, 128), (1, 2, 264, 64), (1, 1, 328, 32)])
def test_attention_matmul_backward_long_sequences(M, B, H, N, Dh, dtype):
    """Long aligned sequences of one to three heads (the kernel for few heads; with more heads these lengths go by tiles: test_gpu_attention_kernels.py)."""
    _attention_case(M, B, H, N, Dh, dtype)


@pytest.mark.parametrize("B,H,N,Dh", [(2, 3, 19, 8), (2, 3, 197, 64), (1, 2, 65, 40), (2, 2, 49, 32)])
def test_attention_matmul_backward_binary32(M, B, H, N, Dh):
    """The same products on binary32 tensors (three bfloat16 parts of each value), to the binary32 bound."""
    _attention_case(M, B, H, N, Dh, torch.float32)


@pytest.mark.parametrize("dtype", [torch.float32, torch.float16, torch.bfloat16], ids=["f32", "f16", "bf16"])
@pytest.mark.parametrize("B,H,N,Dh", [(2, 3, 3, 5), (1, 2, 7, 64), (2, 1, 40, 4), (1, 1, 1, 1)])
def test_attention_matmul_backward_short_extents(M, B, H, N, Dh, dtype):
    """Sequences or heads shorter than one load vector (the plain kernel, in every type)."""
    _attention_case(M, B, H, N, Dh, dtype)


def _mid_of_frame(t, fill):
    """A copy of t in the middle of a larger buffer whose 256 elements on either side hold `fill`."""
    buf = torch.full((t.numel() + 512,), fill, dtype=t.dtype, device=t.device)
    view = buf[256:256 + t.numel()].view(t.shape)
    view.copy_(t)
    return view


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16], ids=["f16", "bf16"])
@pytest.mark.parametrize("B,H,N,Dh", [(1, 2, 197, 64), (2, 1, 49, 32), (1, 2, 64, 64), (1, 1, 128, 64), (1, 1, 200, 64), (1, 1, 256, 64),
                                      (1, 1, 264, 64), (1, 1, 272, 32), (1, 1, 577, 64), (1, 2, 33, 48), (1, 1, 100, 128), (1, 3, 223, 96)])
def test_attention_matmul_backward_uses_nothing_from_outside_its_inputs(M, B, H, N, Dh, dtype):
    """Every input is the middle of a buffer framed by NaN (gradients) or the extreme code: vectors moved back into the
    tensor, clamped loads and masked lanes must not let a value from beyond a tensor's ends into a result."""
    gen = torch.Generator(device="cuda").manual_seed(N * 7 + Dh)
    n2, nd = B * H * N * N, B * H * N * Dh
    ca = _mid_of_frame(torch.randint(-128, 128, (n2,), dtype=torch.int8, device="cuda", generator=gen), 127)
    cq, ck, cvv = (_mid_of_frame(torch.randint(-128, 128, (nd,), dtype=torch.int8, device="cuda", generator=gen), -128) for _ in range(3))
    dO = _mid_of_frame(torch.randn((B, H, N, Dh), device="cuda", generator=gen).to(dtype), float("nan"))
    dS = _mid_of_frame((torch.randn((B, H, N, N), device="cuda", generator=gen) * 0.1).to(dtype), float("nan"))
    par = [(0.5 + torch.rand(H, device="cuda", generator=gen), -0.5 * torch.rand(H, device="cuda", generator=gen)) for _ in range(4)]
    dA = torch.empty((B, H, N, N), dtype=dtype, device="cuda")
    dV, dQ, dK = (torch.empty((B, H, N, Dh), dtype=dtype, device="cuda") for _ in range(3))
    scale = Dh ** -0.5
    M.mesa_attn_av_bwd_q(ca, cvv, B, H, N, Dh, *par[0], *par[1], dO, dA, dV)
    M.mesa_attn_qk_bwd_q(cq, ck, B, H, N, Dh, *par[2], *par[3], dS, scale, dQ, dK)
    rp = [(npy(a), npy(b)) for a, b in par]
    rdA, rdV = R.attn_av_bwd_q(npy(ca), npy(cvv), B, H, N, Dh, *rp[0], *rp[1], npy(dO))
    rdQ, rdK = R.attn_qk_bwd_q(npy(cq), npy(ck), B, H, N, Dh, *rp[2], *rp[3], npy(dS), scale)
    for name, got, ref in (("dA", dA, rdA), ("dV", dV, rdV), ("dQ", dQ, rdQ), ("dK", dK, rdK)):
        g = npy(got)
        assert np.all(np.isfinite(g)), name
        assert relerr(g.reshape(ref.shape), ref) <= TOL[dtype], (name, relerr(g.reshape(ref.shape), ref))


def _attention_case(M, B, H, N, Dh, dtype):
    gen = torch.Generator(device="cuda").manual_seed(B * 1000 + N)
    sig = torch.linspace(0.5, 2.0, H, device="cuda").view(1, H, 1, 1)
    q, k, v = ((torch.randn((B, H, N, Dh), generator=gen, device="cuda") * sig + 0.1 * i).to(dtype).contiguous() for i in range(3))
    scale = Dh ** -0.5
    attn = torch.softmax((q.float() @ k.float().transpose(-1, -2)) * scale, dim=-1).to(dtype).contiguous()
    codes, par, rcodes, rpar = {}, {}, {}, {}
    for name, t, inner in (("q", q, N * Dh), ("k", k, N * Dh), ("v", v, N * Dh), ("a", attn, N * N)):
        lay = (B, H, inner)
        a_, b_, ra, rb = run_params(M, [t], lay)
        c = torch.empty(t.numel(), dtype=torch.int8, device="cuda")
        M.mesa_quantize_headwise(t, lay, a_, b_, c, M.ROUND_STOCHASTIC, 11, 0)
        codes[name], par[name], rcodes[name], rpar[name] = c, (a_, b_), npy(c), (ra, rb)
    dO = torch.randn((B, H, N, Dh), generator=gen, device="cuda").to(dtype)
    dA = torch.empty((B, H, N, N), dtype=dtype, device="cuda")
    dV = torch.empty_like(dO)
    M.mesa_attn_av_bwd_q(codes["a"], codes["v"], B, H, N, Dh, *par["a"], *par["v"], dO, dA, dV)
    rdA, rdV = R.attn_av_bwd_q(rcodes["a"], rcodes["v"], B, H, N, Dh, *rpar["a"], *rpar["v"], npy(dO))
    rep = {"dA": relerr(npy(dA), rdA), "dV": relerr(npy(dV), rdV)}
    dS = torch.empty_like(dA)
    M.mesa_softmax_bwd_q(codes["a"], B, H, N, N, *par["a"], dA, dS)
    dQ = torch.empty_like(dO)
    dK = torch.empty_like(dO)
    M.mesa_attn_qk_bwd_q(codes["q"], codes["k"], B, H, N, Dh, *par["q"], *par["k"], dS, scale, dQ, dK)
    rdQ, rdK = R.attn_qk_bwd_q(rcodes["q"], rcodes["k"], B, H, N, Dh, *rpar["q"], *rpar["k"], npy(dS), scale)
    rep["dQ"], rep["dK"] = relerr(npy(dQ), rdQ), relerr(npy(dK), rdK)
    assert all(v <= TOL[dtype] for v in rep.values()), rep


@pytest.mark.parametrize("dtype", DTYPES, ids=DTYPE_IDS)
@pytest.mark.parametrize("layout", [(3, 4, 1000), (5, 3, 361), (37, 6, 64), (64, 3, 2401), (1, 1, 77)])
def test_symmetric_range_update_matches_the_oracle_bit_for_bit(M, layout, dtype):
    """Symmetric-range running estimates (Sec. 5.2 ablation): first call and two EMA steps, then the codes
    taken with them."""
    G = layout[1]
    gen = torch.Generator(device="cuda").manual_seed(layout[0] * 31 + layout[2])
    xs = [((torch.randn(layout, generator=gen, device="cuda") * (1 + t) + 0.4 * t - 0.3).to(dtype)).contiguous() for t in range(3)]
    a = torch.full((G,), 5.0, device="cuda")
    b = torch.full((G,), -2.0, device="cuda")
    ra, rb = np.full(G, 5.0, np.float32), np.full(G, -2.0, np.float32)
    ws = ws_for(M, M.OP_UPDATE_RUNNING_PARAMS, *layout, dt=dtype)
    for t, x in enumerate(xs):
        M.mesa_update_running_params_sym(x, layout, a, b, 0.9, t == 0, ws)
        ra, rb = R.update_running_params_sym(npy(x), layout, ra, rb, 0.9, t == 0)
        assert np.array_equal(npy(a), ra) and np.array_equal(npy(b), rb), t
    q = torch.empty(xs[-1].numel(), dtype=torch.int8, device="cuda")
    M.mesa_quantize_headwise(xs[-1], layout, a, b, q, M.ROUND_STOCHASTIC, 5, 3)
    rq = R.quantize_headwise(npy(xs[-1]), layout, ra, rb, R.ROUND_STOCHASTIC, 5, 3).reshape(-1)
    assert np.array_equal(npy(q), rq)


@pytest.mark.parametrize("dtype", DTYPES, ids=DTYPE_IDS)
@pytest.mark.parametrize("layout", [(4, 3, 16 * 14 * 14), (5, 3, 361), (3, 40, 77), (1, 1, 1000)])
def test_relu_backward_is_the_oracles_mask_exactly(M, layout, dtype):
    """ReLU backward at group-wise codes (an (N, C, H, W) activation as (N, G, C/G*H*W)); the 0/1 decision is
    taken on the same separately rounded x_hat on both sides, so the result is dy or 0 bit for bit.
    40 groups exceed the table's capacity and take the per-element path."""
    gen = torch.Generator(device="cuda").manual_seed(layout[1] * 7 + layout[2])
    x = (torch.randn(layout, generator=gen, device="cuda") * 1.3 + 0.2).to(dtype).contiguous()
    a, b, ra, rb = run_params(M, [x], layout)
    q = torch.empty(x.numel(), dtype=torch.int8, device="cuda")
    M.mesa_quantize_headwise(x, layout, a, b, q, M.ROUND_STOCHASTIC, 3, 0)
    dy = torch.randn(layout, generator=gen, device="cuda").to(dtype)
    dx = torch.empty_like(dy)
    M.mesa_relu_bwd_q(q, layout, a, b, dy, dx)
    ref = R.relu_bwd_q(npy(q), layout, ra, rb, npy(dy))
    got = npy(dx).astype(np.float64).reshape(ref.shape)
    assert np.array_equal(got, ref)
    frac = float((ref != 0).mean())
    assert 0.2 < frac < 0.8, frac


@pytest.mark.parametrize("dtype", DTYPES, ids=DTYPE_IDS)
@pytest.mark.parametrize("layout", [(37, 6, 256), (5, 3, 361), (64, 12, 128)])
def test_fixed_offset_update_matches_the_oracle_bit_for_bit(M, layout, dtype):
    """Fixed beta = GELU's minimum (Sec. 6) on a GELU-output-like tensor: three steps, then the codes."""
    G = layout[1]
    bf = -0.17
    gen = torch.Generator(device="cuda").manual_seed(layout[0] + 13 * layout[2])
    xs = [torch.nn.functional.gelu(torch.randn(layout, generator=gen, device="cuda") * (1.5 + t)).to(dtype).contiguous() for t in range(3)]
    a = torch.full((G,), 5.0, device="cuda")
    b = torch.full((G,), 9.0, device="cuda")
    ra = np.full(G, 5.0, np.float32)
    ws = ws_for(M, M.OP_UPDATE_RUNNING_PARAMS, *layout, dt=dtype)
    for t, x in enumerate(xs):
        M.mesa_update_running_params_fixed_beta(x, layout, a, b, 0.9, t == 0, bf, ws)
        ra, rb = R.update_running_params_fixed_beta(npy(x), layout, ra, 0.9, t == 0, bf)
        assert np.array_equal(npy(a), ra) and np.array_equal(npy(b), rb), t
    q = torch.empty(xs[-1].numel(), dtype=torch.int8, device="cuda")
    M.mesa_quantize_headwise(xs[-1], layout, a, b, q, M.ROUND_STOCHASTIC, 9, 1)
    rq = R.quantize_headwise(npy(xs[-1]), layout, ra, rb, R.ROUND_STOCHASTIC, 9, 1).reshape(-1)
    assert np.array_equal(npy(q), rq)


@pytest.mark.parametrize("dtype", DTYPES, ids=DTYPE_IDS)
@pytest.mark.parametrize("layout", [(37, 6, 256), (5, 3, 361), (3, 40, 77), (1, 1, 1003)])
def test_gelu_layer_forward_in_one_pass(M, layout, dtype):
    """y = gelu(x) within tolerance of the oracle's binary64 GELU; codes of x and the moved estimates bit for bit
    (two steps, both rounding modes)."""
    G = layout[1]
    gen = torch.Generator(device="cuda").manual_seed(layout[0] * 17 + layout[2])
    a = torch.full((G,), 7.0, device="cuda")
    b = torch.full((G,), -3.5, device="cuda")
    ra, rb = np.full(G, 7.0, np.float32), np.full(G, -3.5, np.float32)
    ws = ws_for(M, M.OP_UPDATE_RUNNING_PARAMS, *layout, dt=dtype)
    for t, (mode, rmode) in enumerate(((M.ROUND_STOCHASTIC, R.ROUND_STOCHASTIC), (M.ROUND_NEAREST_EVEN, R.ROUND_NEAREST))):
        x = (torch.randn(layout, generator=gen, device="cuda") * (1.5 + t)).to(dtype).contiguous()
        y = torch.empty_like(x)
        q = torch.empty(x.numel(), dtype=torch.int8, device="cuda")
        M.mesa_gelu_fwd_q(x, layout, a, b, 0.9, y, q, ws, mode, 21, 4)
        ry, rq, ra, rb = R.gelu_fwd_q(npy(x), layout, ra, rb, 0.9, rmode, 21, 4)
        assert np.array_equal(npy(q), rq.reshape(-1))
        assert np.array_equal(npy(a), ra) and np.array_equal(npy(b), rb)
        assert relerr(npy(y), ry) <= TOL[dtype]


@pytest.mark.parametrize("dtype", DTYPES, ids=DTYPE_IDS)
@pytest.mark.parametrize("B,H,rows,cols", [(3, 6, 197, 197), (5, 3, 49, 49), (2, 4, 64, 64), (1, 2, 33, 1000), (2, 3, 7, 19), (1, 1, 5, 8),
                                           (2, 2, 9, 3), (1, 3, 11, 57), (2, 1, 13, 104), (1, 2, 30, 105), (3, 1, 5, 200), (1, 2, 17, 201),
                                           (2, 2, 6, 256), (1, 2, 10, 257), (40, 3, 61, 61), (1, 1, 3, 4096),
                                           (1, 2, 5, 1025), (1, 1, 3, 4097), (2, 1, 2, 9001), (1, 1, 2, 8200), (1, 1100, 2, 300),
                                           (2, 2, 9, 57), (1, 3, 8, 63), (2, 1, 5, 105), (1, 2, 6, 128), (1, 1, 7, 120),
                                           # more long rows of 8k elements, and tiles that change heads on the way
                                           (1, 2, 5, 264), (2, 2, 4, 512), (1, 2, 4, 520), (1, 2, 6, 768), (1, 1, 3, 1024), (1, 2, 2, 1032),
                                           (1, 1, 3, 1536), (1, 1, 3, 2048), (1, 1, 2, 2056), (2, 3, 4400, 264), (1, 2, 9000, 520)])
def test_softmax_backward_every_row_shape(M, B, H, rows, cols, dtype):
    """Softmax backward at head-wise codes over every lane-group shape of the short-row kernel (and both of its
    variants), rows shorter than a vector, ragged tiles, tiles that straddle heads, and the long-row kernel; the plain
    kernel's shapes (odd rows above 1024 elements, rows above 8192, more than 1024 heads); out of place and in place."""
    gen = torch.Generator(device="cuda").manual_seed(B * 10 + cols)
    lay = (B, H, rows * cols)
    sig = torch.linspace(0.5, 3.0, H, device="cuda").view(1, H, 1, 1)
    y = torch.softmax(torch.randn((B, H, rows, cols), generator=gen, device="cuda") * sig, dim=-1).to(dtype).contiguous()
    a, b, ra, rb = run_params(M, [y], lay)
    q = torch.empty(y.numel(), dtype=torch.int8, device="cuda")
    M.mesa_quantize_headwise(y, lay, a, b, q, M.ROUND_STOCHASTIC, 5, 0)
    dy = torch.randn((B, H, rows, cols), generator=gen, device="cuda").to(dtype)
    dx = torch.empty_like(dy)
    M.mesa_softmax_bwd_q(q, B, H, rows, cols, a, b, dy, dx)
    ref = R.softmax_bwd_q(npy(q), B, H, rows, cols, ra, rb, npy(dy))
    assert relerr(npy(dx).reshape(ref.shape), ref) <= TOL[dtype]
    dy2 = dy.clone()
    M.mesa_softmax_bwd_q(q, B, H, rows, cols, a, b, dy2, dy2)
    assert torch.equal(dy2, dx)


@pytest.mark.parametrize("dtype", DTYPES, ids=DTYPE_IDS)
@pytest.mark.parametrize("B,H,rows,cols", [(3, 6, 197, 197), (5, 3, 49, 49), (2, 4, 64, 64), (1, 2, 33, 1000), (2, 3, 7, 19), (1, 1, 5, 8),
                                           (2, 2, 9, 3), (1, 3, 11, 57), (2, 1, 13, 104), (1, 2, 30, 105), (3, 1, 5, 200), (1, 2, 17, 201),
                                           (2, 2, 6, 256), (1, 2, 10, 257), (40, 3, 61, 61),
                                           (2, 2, 9, 57), (1, 3, 8, 63), (2, 1, 5, 105), (1, 2, 6, 128), (1, 1, 7, 120),
                                           # rows of 8k elements beyond 256: a wave per row, one to eight vectors per lane
                                           (1, 2, 5, 264), (2, 2, 3, 512), (1, 2, 4, 520), (1, 1, 3, 1024), (1, 2, 2, 1032),
                                           (1, 1, 3, 2048), (1, 1, 2, 2056), (1, 2, 2, 4096), (1, 1, 2, 4104),
                                           # ... whose waves walk several rows and change heads on the way
                                           (2, 3, 700, 264), (1, 2, 1100, 2056),
                                           # what no single-pass kernel takes: a plain softmax, then the single-pass quantizer on y
                                           (1, 2, 3, 3001), (2, 1, 5, 1025), (2, 1500, 3, 19), (1, 3, 2, 8200), (1, 6000, 2, 24)])
def test_softmax_layer_forward_in_one_pass(M, B, H, rows, cols, dtype):
    """y = softmax(s) within tolerance of the oracle's binary64 softmax and with rows that sum to 1; the codes and
    the moved estimates are exactly the oracle's single-pass forward applied to the y the kernel stored
    (the decision is taken on the stored value on both sides); two steps, both rounding modes."""
    gen = torch.Generator(device="cuda").manual_seed(B * 100 + cols)
    lay = (B, H, rows * cols)
    a = torch.full((H,), 0.9, device="cuda")
    b = torch.full((H,), 0.01, device="cuda")
    ws = torch.empty(max(M.workspace_bytes(M.OP_SOFTMAX_FWD_Q, B * H * rows, H, cols, M.F16), 16), dtype=torch.uint8, device="cuda")
    sig = torch.linspace(0.5, 3.0, H, device="cuda").view(1, H, 1, 1)
    for t, (mode, rmode) in enumerate(((M.ROUND_STOCHASTIC, R.ROUND_STOCHASTIC), (M.ROUND_NEAREST_EVEN, R.ROUND_NEAREST))):
        s = (torch.randn((B, H, rows, cols), generator=gen, device="cuda") * sig * (1 + t)).to(dtype).contiguous()
        y = torch.empty_like(s)
        q = torch.empty(s.numel(), dtype=torch.int8, device="cuda")
        ra, rb = npy(a).copy(), npy(b).copy()
        M.mesa_softmax_fwd_q(s, B, H, rows, cols, a, b, 0.9, y, q, ws, mode, 31, 7)
        yh = npy(y)
        ref = R.softmax_fwd(npy(s), B * H * rows, cols)
        assert relerr(yh, ref) <= TOL[dtype]
        assert np.abs(yh.astype(np.float64).sum(-1) - 1.0).max() <= TOL[dtype]
        rq, ra2, rb2 = R.quantize_update_fused(yh, lay, ra, rb, 0.9, rmode, 31, 7)
        assert np.array_equal(npy(q), rq.reshape(-1))
        assert np.array_equal(canon(npy(a)), canon(ra2)) and np.array_equal(canon(npy(b)), canon(rb2))


@pytest.mark.parametrize("dtype", DTYPES, ids=DTYPE_IDS)
@pytest.mark.parametrize("Mr,D,G", [(1000, 384, 6), (77, 768, 12), (50, 1024, 4), (33, 64, 2), (19, 8, 1), (300, 96, 3), (5, 520, 1),
                                    (41, 1032, 3), (130, 1536, 12), (9, 2048, 16),
                                    # what the single-pass kernel does not take: plain statistics and y, then the single-pass quantizer on x
                                    (6, 84, 7), (4, 4096, 8), (3, 5000, 5), (10, 96, 24), (3, 3000, 1500)])
def test_layernorm_layer_forward_in_one_pass(M, Mr, D, G, dtype):
    """y, mean and rstd within tolerance of the oracle's binary64 LayerNorm; codes of x and the moved estimates bit
    for bit (two steps, both rounding modes); the statistics feed the backward call as they are."""
    gen = torch.Generator(device="cuda").manual_seed(Mr * 7 + D)
    lay = (Mr, G, D // G)
    a = torch.full((G,), 9.0, device="cuda")
    b = torch.full((G,), -4.5, device="cuda")
    ra, rb = np.full(G, 9.0, np.float32), np.full(G, -4.5, np.float32)
    gamma = (1 + 0.1 * torch.randn(D, generator=gen, device="cuda")).to(dtype)
    bias = (0.1 * torch.randn(D, generator=gen, device="cuda")).to(dtype)
    ws = torch.empty(max(M.workspace_bytes(M.OP_LAYERNORM_FWD_Q, Mr, D, G, M.F16), 16), dtype=torch.uint8, device="cuda")
    for t, (mode, rmode) in enumerate(((M.ROUND_STOCHASTIC, R.ROUND_STOCHASTIC), (M.ROUND_NEAREST_EVEN, R.ROUND_NEAREST))):
        x = ((torch.randn((Mr, D), generator=gen, device="cuda") * (1.0 + t) + 0.3)).to(dtype).contiguous()
        y = torch.empty_like(x)
        mean = torch.empty(Mr, device="cuda")
        rstd = torch.empty(Mr, device="cuda")
        q = torch.empty(x.numel(), dtype=torch.int8, device="cuda")
        M.mesa_layernorm_fwd_q(x, Mr, D, G, gamma, bias, 1e-5, a, b, 0.9, y, mean, rstd, q, ws, mode, 13, 5)
        ry, rmean, rrstd = R.layernorm_fwd(npy(x), Mr, D, npy(gamma), npy(bias), 1e-5)
        assert relerr(npy(y), ry) <= TOL[dtype]
        assert relerr(npy(mean), rmean) <= 1e-5 and relerr(npy(rstd), rrstd) <= 1e-5
        rq, ra, rb = R.quantize_update_fused(npy(x), lay, ra, rb, 0.9, rmode, 13, 5)
        assert np.array_equal(npy(q), rq.reshape(-1))
        assert np.array_equal(canon(npy(a)), canon(ra)) and np.array_equal(canon(npy(b)), canon(rb))


def test_empty_inputs_are_a_no_op(M):
    z = torch.empty(0, device="cuda")
    a = torch.ones(3, device="cuda")
    b = torch.zeros(3, device="cuda")
    q = torch.empty(0, dtype=torch.int8, device="cuda")
    ws = torch.empty(16, dtype=torch.uint8, device="cuda")
    M.mesa_update_running_params(z, (0, 3, 5), a, b, 0.9, True, ws)
    M.mesa_quantize_headwise(z, (0, 3, 5), a, b, q)
    M.mesa_dequantize(q, (0, 3, 5), a, b, z)
    M.mesa_gelu_bwd_q(q, (0, 3, 5), a, b, z, z)
    M.mesa_softmax_bwd_q(q, 0, 3, 4, 8, a, b, z, z)
    torch.cuda.synchronize()
    assert a.cpu().tolist() == [1, 1, 1]


def test_in_place_gradients_and_determinism(M):
    spec = W.small_case(torch.float16, B=4, H=3, N=49, D=96, mlp=384)
    lay = spec.gelu_layout
    x = W.gelu_input(spec, 0, "cuda")
    a = torch.zeros(3, device="cuda"); b = torch.zeros(3, device="cuda")
    ws = ws_for(M, M.OP_UPDATE_RUNNING_PARAMS, *lay)
    M.mesa_update_running_params(x, lay, a, b, 0.9, True, ws)
    q = torch.empty(x.numel(), dtype=torch.int8, device="cuda")
    M.mesa_quantize_headwise(x, lay, a, b, q, M.ROUND_STOCHASTIC, 7, 0)
    q2 = torch.empty_like(q)
    M.mesa_quantize_headwise(x, lay, a, b, q2, M.ROUND_STOCHASTIC, 7, 0)
    assert torch.equal(q, q2)
    dy = W.upstream_grad(spec, "dy_gelu", x.shape, "cuda")
    dx = torch.empty_like(dy)
    M.mesa_gelu_bwd_q(q, lay, a, b, dy, dx)
    dy2 = dy.clone()
    M.mesa_gelu_bwd_q(q, lay, a, b, dy2, dy2)
    assert torch.equal(dx, dy2)
    # softmax in place
    Bq, Hq, r, c = spec.attn
    y = W.attention_map(spec, 0, "cuda")
    M.mesa_update_running_params(y, spec.attn_layout, a, b, 0.9, True, ws_for(M, M.OP_UPDATE_RUNNING_PARAMS, *spec.attn_layout))
    qa = torch.empty(y.numel(), dtype=torch.int8, device="cuda")
    M.mesa_quantize_headwise(y, spec.attn_layout, a, b, qa, M.ROUND_NEAREST_EVEN)
    dya = W.upstream_grad(spec, "dy_attn", y.shape, "cuda")
    dxa = torch.empty_like(dya)
    M.mesa_softmax_bwd_q(qa, Bq, Hq, r, c, a, b, dya, dxa)
    dyb = dya.clone()
    M.mesa_softmax_bwd_q(qa, Bq, Hq, r, c, a, b, dyb, dyb)
    assert torch.equal(dxa, dyb)


@pytest.mark.parametrize("dtype", DTYPES, ids=DTYPE_IDS)
@pytest.mark.parametrize("rows,cols", [(49, 49), (197, 197), (5, 300), (5, 304), (3, 2304)])
def test_softmax_layer_forward_with_masked_logits(M, rows, cols, dtype):
    """Logits of -inf (an attention mask) get probability exactly 0 and do not disturb the rest of their row, in
    the short-row, the long-row and the wave-per-row kernel; rows keep at least one finite logit."""
    B, H = 2, 3
    gen = torch.Generator(device="cuda").manual_seed(rows + cols)
    s = (torch.randn((B, H, rows, cols), generator=gen, device="cuda") * 3).to(dtype)
    mask = torch.rand((B, H, rows, cols), generator=gen, device="cuda") < 0.4
    mask[..., 0] = False
    s = s.masked_fill(mask, float("-inf")).contiguous()
    y = torch.empty_like(s)
    q = torch.empty(s.numel(), dtype=torch.int8, device="cuda")
    a = torch.full((H,), 0.9, device="cuda")
    b = torch.zeros(H, device="cuda")
    ra, rb = npy(a).copy(), npy(b).copy()
    ws = torch.empty(max(M.workspace_bytes(M.OP_SOFTMAX_FWD_Q, B * H * rows, H, cols, M.F16), 16), dtype=torch.uint8, device="cuda")
    M.mesa_softmax_fwd_q(s, B, H, rows, cols, a, b, 0.9, y, q, ws, M.ROUND_STOCHASTIC, 1, 2)
    yh = npy(y)
    assert np.all(yh[npy(mask)] == 0.0) and np.all(np.isfinite(yh))
    assert relerr(yh, R.softmax_fwd(npy(s), B * H * rows, cols)) <= TOL[dtype]
    rq, ra2, rb2 = R.quantize_update_fused(yh, (B, H, rows * cols), ra, rb, 0.9, R.ROUND_STOCHASTIC, 1, 2)
    assert np.array_equal(npy(q), rq.reshape(-1))
    assert np.array_equal(canon(npy(a)), canon(ra2)) and np.array_equal(canon(npy(b)), canon(rb2))


@pytest.mark.parametrize("dtype", DTYPES, ids=DTYPE_IDS)
@pytest.mark.parametrize("scale", [20.0, 3000.0])
def test_softmax_layer_forward_with_large_logits(M, scale, dtype):
    """Logits far from zero (nearly one-hot rows): the maximum is subtracted before the exponential, so the result
    keeps its accuracy, in the short-row and in the long-row kernel."""
    for cols in (49, 197, 300, 320):
        B, H, rows = 2, 3, 33
        gen = torch.Generator(device="cuda").manual_seed(int(scale) + cols)
        s = (torch.randn((B, H, rows, cols), generator=gen, device="cuda") * scale).to(dtype).contiguous()
        y = torch.empty_like(s)
        q = torch.empty(s.numel(), dtype=torch.int8, device="cuda")
        a = torch.full((H,), 0.9, device="cuda")
        b = torch.zeros(H, device="cuda")
        ws = torch.empty(max(M.workspace_bytes(M.OP_SOFTMAX_FWD_Q, B * H * rows, H, cols, M.F16), 16), dtype=torch.uint8, device="cuda")
        M.mesa_softmax_fwd_q(s, B, H, rows, cols, a, b, 0.9, y, q, ws, M.ROUND_NEAREST_EVEN, 0, 0)
        assert relerr(npy(y), R.softmax_fwd(npy(s), B * H * rows, cols)) <= TOL[dtype], (cols, scale)


@pytest.mark.parametrize("dtype", [torch.float16, torch.float32], ids=["f16", "f32"])
@pytest.mark.parametrize("layout", [(3, 3000, 40), (2, 4096, 16), (1, 8192, 24), (5, 700, 361)])
def test_thousands_of_groups(M, layout, dtype):
    """Per-sample statistics of a large batch are thousands of groups: the parameter tables and the per-group
    extrema then fill most of a workgroup's local memory.  Update, quantize, de-quantize and GELU backward up to
    the limit of 8192 groups (the single-pass forward beyond 4096 with more local memory than a launch gets by default)."""
    outer, G, inner = layout
    n = outer * G * inner
    gen = torch.Generator(device="cuda").manual_seed(G + inner)
    scale = (0.2 + 3.0 * torch.rand((1, G, 1), generator=gen, device="cuda"))
    xs = [((torch.randn(layout, generator=gen, device="cuda") * scale) + 0.1 * t).to(dtype).contiguous() for t in range(2)]
    a, b, ra, rb = run_params(M, xs, layout)
    assert np.array_equal(canon(npy(a)), canon(ra)) and np.array_equal(canon(npy(b)), canon(rb))
    x = xs[-1]
    q = torch.empty(n, dtype=torch.int8, device="cuda")
    M.mesa_quantize_headwise(x, layout, a, b, q, M.ROUND_STOCHASTIC, 9, 1)
    rq = R.quantize_headwise(npy(x), layout, ra, rb, R.ROUND_STOCHASTIC, 9, 1).reshape(-1)
    assert np.array_equal(npy(q), rq)
    xh = torch.empty(n, dtype=dtype, device="cuda")
    M.mesa_dequantize(q, layout, a, b, xh)
    u = np.uint32 if dtype == torch.float32 else np.uint16
    assert np.array_equal(npy(xh).view(u), R.dequantize(rq, layout, ra, rb, np.float32 if dtype == torch.float32 else np.float16).view(u).reshape(-1))
    dy = torch.randn(layout, generator=gen, device="cuda").to(dtype)
    dx = torch.empty_like(dy)
    M.mesa_gelu_bwd_q(q, layout, a, b, dy, dx)
    assert relerr(npy(dx).reshape(-1), R.gelu_bwd_q(rq, layout, ra, rb, npy(dy)).reshape(-1)) <= TOL[dtype]
    # the single-pass forward on the same tensor
    a2, b2 = a.clone(), b.clone()
    q2 = torch.empty(n, dtype=torch.int8, device="cuda")
    ws = ws_for(M, M.OP_UPDATE_RUNNING_PARAMS, *layout, dt=dtype)
    M.mesa_quantize_update_fused(x, layout, a2, b2, 0.9, q2, ws, M.ROUND_STOCHASTIC, 9, 1)
    rq2, ra2, rb2 = R.quantize_update_fused(npy(x), layout, ra, rb, 0.9, R.ROUND_STOCHASTIC, 9, 1)
    assert np.array_equal(npy(q2), rq2.reshape(-1))
    assert np.array_equal(canon(npy(a2)), canon(ra2)) and np.array_equal(canon(npy(b2)), canon(rb2))


@pytest.mark.parametrize("mean", [0.0, 0.5])
def test_linear_dw_upstream_gradient_with_a_mean(M, mean):
    """The binary16 weight gradient contracts dy with 1024 + x_bar (the constant is taken out again with the row
    sums), so the binary32 sums carry a term 1024 * sum(dy) that the result does not: with an upstream gradient whose
    mean is far from zero AND a de-quantized input centred on zero the cancellation is at its worst.  Half a standard
    deviation of mean over 20000 rows must stay well inside the 2e-3 bound (measured: 3e-4 at 50000 rows)."""
    Mr, K, N, G = 20000, 256, 512, 4
    gen = torch.Generator(device="cuda").manual_seed(7)
    q = torch.randint(-128, 128, (Mr, K), dtype=torch.int8, device="cuda", generator=gen)
    dy = (torch.randn((Mr, N), device="cuda", generator=gen) + mean).half()
    a = torch.full((G,), 8.0, device="cuda")
    b = torch.full((G,), -4.0, device="cuda")     # x_hat in [-4, 4]
    dW = torch.empty((N, K), device="cuda")
    db = torch.empty(N, device="cuda")
    ws = ws_for(M, M.OP_LINEAR_DW_Q, Mr, K, N, torch.float16)
    M.mesa_linear_dw_q(q, Mr, K, G, a, b, dy, N, dW, db, ws)
    rW, rb = R.linear_dw_q(npy(q), Mr, K, G, npy(a), npy(b), npy(dy), N)
    assert relerr(npy(dW), rW) <= 5e-4, relerr(npy(dW), rW)
    assert relerr(npy(db), rb) <= 1e-5


@pytest.mark.parametrize("dtype", DTYPES, ids=DTYPE_IDS)
@pytest.mark.parametrize("layout", [(3, 4, 1000), (5, 3, 361), (37, 6, 64), (1, 1, 12345), (7, 5, 3), (3000, 12, 256)])
def test_scale_only_symmetric_scheme_is_bit_exact(M, layout, dtype):
    """The ablation's comparison scheme (Sec. 5.2): running scale after a first call and two moving-average steps,
    codes in both rounding modes and the de-quantized values, all bit for bit against the oracle; and the fused GELU
    backward fed with these codes through the equivalent (alpha, beta) pair."""
    outer, G, inner = layout
    n = outer * G * inner
    gen = torch.Generator(device="cuda").manual_seed(n + 5)
    scale = torch.tensor([0.3, 1.0, 4.0, 11.0, 0.05, 2.0, 7.0, 1.5, 0.8, 3.0, 0.1, 6.0], device="cuda")[:G].view(1, G, 1)
    xs = [(torch.randn((outer, G, inner), generator=gen, device="cuda") * scale * (1.0 + 0.3 * i) - 0.2 * i).to(dtype).contiguous()
          for i in range(3)]
    m = torch.full((G,), 9.0, device="cuda")
    rm = np.full(G, 9.0, np.float32)
    ws = ws_for(M, M.OP_UPDATE_RUNNING_PARAMS, *layout, dt=dtype)
    for i, x in enumerate(xs):
        M.mesa_update_running_scale_sym(x, layout, m, 0.9, i == 0, ws)
        rm = R.update_running_scale_sym(npy(x), layout, rm, 0.9, i == 0)
        assert np.array_equal(canon(npy(m)), canon(rm)), i
    x = xs[-1]          # the running scale lags the last batch: some elements saturate
    for mode, seed, off in ((M.ROUND_NEAREST_EVEN, 0, 0), (M.ROUND_STOCHASTIC, 0xABCDEF0123, (1 << 34) + 3)):
        q = torch.empty(n, dtype=torch.int8, device="cuda")
        M.mesa_quantize_sym(x, layout, m, q, mode, seed, off)
        rq = R.quantize_sym(npy(x), layout, rm, mode, seed, off).reshape(-1)
        bad = np.nonzero(npy(q) != rq)[0]
        assert bad.size == 0, (mode, bad[:10], npy(q)[bad[:10]], rq[bad[:10]])
        assert int(q.min()) >= -127
    for odt, npo, u in ((torch.float32, np.float32, np.uint32), (torch.float16, np.float16, np.uint16)):
        out = torch.empty(n, dtype=odt, device="cuda")
        M.mesa_dequantize_sym(q, layout, m, out)
        assert np.array_equal(npy(out).view(u), R.dequantize_sym(rq, layout, rm, npo).view(u))
    out = torch.empty(n, dtype=torch.bfloat16, device="cuda")
    M.mesa_dequantize_sym(q, layout, m, out)
    assert np.array_equal(out.view(torch.int16).cpu().numpy().view(np.uint16), R.dequantize_sym(rq, layout, rm, "bf16").reshape(-1))
    # backward through the asymmetric form of the same reconstruction
    a_eq, b_eq = m * (255.0 / 127.0), m * (-128.0 / 127.0)
    dy = torch.randn((outer, G, inner), generator=gen, device="cuda").to(dtype)
    dx = torch.empty_like(dy)
    M.mesa_gelu_bwd_q(q, layout, a_eq, b_eq, dy, dx)
    ref = R.gelu_bwd_q(rq, layout, npy(a_eq), npy(b_eq), npy(dy)).reshape(-1)
    assert relerr(npy(dx).reshape(-1), ref) <= TOL[dtype]
    # and that pair does reproduce the symmetric reconstruction, to rounding
    xa = R.dequantize(rq, layout, npy(a_eq), npy(b_eq), np.float32).astype(np.float64)
    xsym = R.dequantize_sym(rq, layout, rm, np.float32).astype(np.float64)
    assert np.abs(xa - xsym).max() <= 4e-6 * max(float(rm.max()), 1e-30)


@pytest.mark.parametrize("dtype", DTYPES, ids=DTYPE_IDS)
@pytest.mark.parametrize("layout", [(3, 4, 1000), (5, 3, 361), (37, 6, 64), (1, 1, 12345), (7, 5, 3), (1, 1, 5), (3000, 12, 256),
                                    (3, 2000, 40)])
def test_four_bit_codes_are_bit_exact(M, layout, dtype):
    """Four-bit codes (fifteen steps, two codes per byte): packed codes in both rounding modes and the de-quantized
    values bit for bit against the oracle -- odd element counts, slabs shorter than a vector, nibble pairs that
    straddle groups, more groups than the gradient table holds -- and the GELU backward within tolerance."""
    outer, G, inner = layout
    n = outer * G * inner
    gen = torch.Generator(device="cuda").manual_seed(n + 11)
    scale = (0.3 + 3.0 * torch.rand((1, G, 1), generator=gen, device="cuda"))
    xs = [((torch.randn((outer, G, inner), generator=gen, device="cuda") * scale) + 0.2 * i).to(dtype).contiguous() for i in range(2)]
    a, b, ra, rb = run_params(M, xs, layout)
    x = xs[-1]
    nb = (n + 1) // 2
    for mode, seed, off in ((M.ROUND_NEAREST_EVEN, 0, 0), (M.ROUND_STOCHASTIC, 0xFEED5EED, (1 << 33) + 5)):
        q4 = torch.full((nb + 16,), 0xAB, dtype=torch.uint8, device="cuda")     # sentinel bytes behind the codes
        M.mesa_quantize_headwise_b4(x, layout, a, b, q4, mode, seed, off)
        rq4 = R.quantize_headwise_b4(npy(x), layout, ra, rb, mode, seed, off)
        got = q4.cpu().numpy()
        bad = np.nonzero(got[:nb] != rq4)[0]
        assert bad.size == 0, (mode, bad[:10], got[bad[:10]], rq4[bad[:10]])
        assert np.all(got[nb:] == 0xAB)
    q4 = q4[:nb].clone()
    for odt, npo, u in ((torch.float32, np.float32, np.uint32), (torch.float16, np.float16, np.uint16)):
        out = torch.empty(n, dtype=odt, device="cuda")
        M.mesa_dequantize_b4(q4, layout, a, b, out)
        assert np.array_equal(npy(out).view(u), R.dequantize_b4(rq4, layout, ra, rb, npo).view(u))
    out = torch.empty(n, dtype=torch.bfloat16, device="cuda")
    M.mesa_dequantize_b4(q4, layout, a, b, out)
    assert np.array_equal(out.view(torch.int16).cpu().numpy().view(np.uint16), R.dequantize_b4(rq4, layout, ra, rb, "bf16"))
    dy = torch.randn((outer, G, inner), generator=gen, device="cuda").to(dtype)
    dx = torch.empty_like(dy)
    M.mesa_gelu_bwd_q_b4(q4, layout, a, b, dy, dx)
    ref = R.gelu_bwd_q_b4(rq4, layout, ra, rb, npy(dy))
    assert relerr(npy(dx).reshape(-1), ref) <= TOL[dtype]
    M.mesa_gelu_bwd_q_b4(q4, layout, a, b, dy, dy)          # in place
    assert torch.equal(dy, dx)
