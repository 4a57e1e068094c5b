"""The work that a training program has libmesa do, as cases that can be prepared, run and timed.

A case is a dict of plain values: `kind` says which public calls it makes, `dtype` the storage type of activations and
gradients, `stochastic` the rounding of the codes, and the rest are sizes. The kinds:

  saved      one saved tensor through the two-call forward (running estimates, then codes) and the de-quantizer
  softmax    a softmax layer: the forward that ends in codes of the attention map, and the backward
  gelu       a GELU layer: the forward that ends in codes of the input, and the backward
  layernorm  a LayerNorm layer: the forward that ends in codes of the input, and the backward
  linear     the weight gradient of a Linear layer at its saved input
  attention  the backward of scaled dot-product attention: the A V product, softmax, the Q K^T product
  conv       the weight gradient of a convolution at its saved input
  block      a whole Transformer block: its eleven saved tensors through the two-call forward, then every backward call

Between a layer's forward and its backward a training step runs all the layers above it, so the backward of a single layer
takes codes that an earlier forward left behind; a block's backward takes the codes of the block's own forward.

Sizes are those of this repository's configurations (mesa_workloads.py), of bench.py's legs and of the tests; distributions
are theirs too. `draw` gives more cases of the same ranges.
"""
from __future__ import annotations

import math

import torch

import paper_2111_11124_amd as m

DEV = "cuda:0"
DTYPES = {"f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32}
MESA_DTYPES = {torch.float16: m.F16, torch.bfloat16: m.BF16, torch.float32: m.F32}
LAM = 0.9
EPS = 1e-5


# ---------------------------------------------------------------------------------------------------------------- cases
def listed():
    return [
        # the smallest calls: a DeiT-Ti block at batch 2 in binary32 -- some fifty launches that each move well under a
        # megabyte, so what is measured is their latency
        dict(name="block_deit_ti_b2_f32", kind="block", dtype="f32", stochastic=True, B=2, N=197, D=192, H=3, mlp=768),
        # an ordinary training step: the whole DeiT-S block at batch 128 in binary16
        dict(name="block_deit_s_b128_f16", kind="block", dtype="f16", stochastic=True, B=128, N=197, D=384, H=6, mlp=1536),
        # the largest head-wise tensor of DeiT-B at batch 256: its attention maps, odd slabs of 197 x 197
        dict(name="saved_map_deit_b_f16", kind="saved", dtype="f16", stochastic=True, outer=256, groups=12, inner=197 * 197),
        # Swin-T's first stage: softmax over windows of 49 tokens, very many short odd rows
        dict(name="softmax_windows_swin_t_f16", kind="softmax", dtype="f16", stochastic=True, B=8192, H=3, N=49),
        # a DeiT-B shape at higher resolution (24 x 24 patches and a class token): long odd rows, bfloat16
        dict(name="softmax_577_bf16", kind="softmax", dtype="bf16", stochastic=True, B=16, H=12, N=577),
        # the widest activation of a DeiT-B block at batch 256: the GELU between its two MLP layers
        dict(name="gelu_deit_b_f16", kind="gelu", dtype="f16", stochastic=True, M=256 * 197, D=3072, G=12),
        # one of the two LayerNorms of that block
        dict(name="layernorm_deit_b_f16", kind="layernorm", dtype="f16", stochastic=True, M=256 * 197, D=768, G=12),
        # the largest weight gradient of that block: its first MLP layer
        dict(name="linear_mlp_deit_b_f16", kind="linear", dtype="f16", M=256 * 197, K=768, G=12, N_out=3072),
        # the QKV layer of a long-sequence block (8 x 4096 tokens, width 1024), bfloat16
        dict(name="linear_qkv_long_bf16", kind="linear", dtype="bf16", M=8 * 4096, K=1024, G=16, N_out=3072),
        # the attention backward of DeiT-S at batch 128: sequences of 197
        dict(name="attention_deit_s_b128_f16", kind="attention", dtype="f16", B=128, H=6, N=197, Dh=64),
        # the attention backward of one long sequence: 4096 tokens, 16 heads, bfloat16
        dict(name="attention_4096_bf16", kind="attention", dtype="bf16", B=1, H=16, N=4096, Dh=64),
        # a 3 x 3 convolution of a segmentation head: 512 channels on 128 x 128 maps
        dict(name="conv3x3_segmentation_f16", kind="conv", dtype="f16", B=2, C_in=512, H=128, W=128, C_out=512, k=3, G=8),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the ranges that the listed ones stand for."""
    kind = rng.choice(["saved", "softmax", "gelu", "layernorm", "linear", "attention", "conv", "block"])
    dtype = rng.choice(["f16", "f16", "f16", "bf16", "bf16", "f32"])
    stochastic = rng.random() < 0.8
    most = 1.1e8 if dtype != "f32" else 5.5e7                # elements of the largest tensor
    if kind == "saved":
        n = _log(rng, 2e4, most)
        groups = rng.choice([1, 2, 3, 4, 6, 8, 12, 16, 24, 32])
        if rng.random() < 0.5:                               # head-wise: long slabs, odd lengths among them
            rows = _log(rng, 14, 1100)
            inner = rows * rng.choice([rows, 32, 64])
        else:                                                # channel groups of a token matrix
            inner = rng.choice([8, 16, 20, 32, 64, 96, 128, 256, 341])
        return dict(kind=kind, dtype=dtype, stochastic=stochastic, outer=max(1, n // (groups * inner)), groups=groups, inner=inner)
    if kind == "softmax":
        n, N = _log(rng, 2e4, most), _log(rng, 16, 2048)
        H = rng.choice([1, 2, 3, 4, 6, 8, 12, 16])
        return dict(kind=kind, dtype=dtype, stochastic=stochastic, B=max(1, n // (H * N * N)), H=H, N=N)
    if kind in ("gelu", "layernorm"):
        n = _log(rng, 2e4, most)
        G = rng.choice([1, 2, 3, 4, 6, 8, 12, 16])
        D = G * 8 * rng.randint(1, 32) if kind == "gelu" else G * 8 * rng.randint(2, 16)
        return dict(kind=kind, dtype=dtype, stochastic=stochastic, M=max(1, n // D), D=D, G=G)
    if kind == "linear":
        G = rng.choice([1, 3, 4, 6, 8, 12, 16])
        K = G * 16 * rng.randint(2, 16)
        N_out = 8 * _log(rng, 8, 512)
        M = _log(rng, 197, 50432)
        M = min(M, int((2.3e11 if dtype != "f32" else 2e10) / (2 * K * N_out)), int(1.5e8 / (K + N_out)))
        return dict(kind=kind, dtype=dtype, M=max(64, M), K=K, G=G, N_out=N_out)
    if kind == "attention":
        N, Dh = _log(rng, 40, 1100), rng.choice([32, 64, 64, 64, 96, 128])
        H = rng.choice([3, 4, 6, 8, 12, 16])
        n = _log(rng, 2e4, 3e7 if dtype != "f32" else 4e6)
        return dict(kind=kind, dtype=dtype, B=max(1, n // (H * N * N)), H=H, N=N, Dh=Dh)
    if kind == "conv":
        dtype = rng.choice(["f16", "bf16"])
        W = rng.randint(7, 128)
        H = max(7, W + rng.choice([0, 0, 0, -4, 5]))
        G = rng.choice([1, 2, 4, 8])
        C_in, C_out, k = G * 8 * rng.randint(2, 8), 16 * rng.randint(2, 32), rng.choice([1, 3, 3])
        B = min(_log(rng, 1, 64), max(1, int(1.5e11 / (2 * k * k * C_in * C_out * H * W))), max(1, int(2e7 / (max(C_in, C_out) * H * W))))
        return dict(kind=kind, dtype=dtype, B=B, C_in=C_in, H=H, W=W, C_out=C_out, k=k, G=G)
    H, Dh = rng.choice([(3, 64), (6, 64), (12, 64), (3, 32), (8, 32)])
    N = _log(rng, 40, 260)
    B = _log(rng, 1, 96) if dtype != "f32" else _log(rng, 1, 8)
    return dict(kind="block", dtype=dtype, stochastic=stochastic, B=max(1, min(B, int(2.4e4 / N))), N=N, D=H * Dh, H=H, mlp=4 * H * Dh)


# --------------------------------------------------------------------------------------------------------------- inputs
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _normal(shape, g, dtype=torch.float32):
    if dtype == torch.float32:
        return torch.randn(shape, generator=g, device=DEV)
    out = torch.empty(shape, dtype=dtype, device=DEV)
    flat = out.view(-1)
    for at in range(0, flat.numel(), 1 << 27):
        n = min(1 << 27, flat.numel() - at)
        flat[at:at + n] = torch.randn(n, generator=g, device=DEV).to(dtype)
    return out


def _tokens(shape, g, dtype):
    """LayerNorm and Linear inputs: N(0, 1) with one element in a thousand twenty times as large."""
    x = _normal(shape, g)
    x = torch.where(torch.rand(shape, generator=g, device=DEV) < 1e-3, 20 * x, x)
    return x.to(dtype)


def _head_sigma(H, g):
    lo, hi = math.log(0.25), math.log(4.0)
    return torch.exp(lo + (hi - lo) * torch.rand(H, generator=g, device=DEV)).view(1, H, 1, 1)


def _logits(B, H, N, g, dtype):
    out = torch.empty((B, H, N, N), dtype=dtype, device=DEV)
    sig = _head_sigma(H, g)
    per = max(1, (1 << 26) // (H * N * N))
    for b in range(0, B, per):
        e = min(B, b + per)
        out[b:e] = torch.randn((e - b, H, N, N), generator=g, device=DEV) * sig
    return out


def _map(B, H, N, g, dtype):
    s = _logits(B, H, N, g, dtype)
    for b in range(B):
        s[b] = torch.softmax(s[b].float(), -1).to(dtype)
    return s


def _estimates(x, L, g):
    """Running estimates of a tensor like x, as training has them: near this batch's extrema and not equal to them."""
    v = x.view(L)
    mn, mx = v.amin(dim=(0, 2)).float(), v.amax(dim=(0, 2)).float()
    r = 0.9 + 0.12 * torch.rand((2, L[1]), generator=g, device=DEV)
    return ((mx - mn) * r[0]).contiguous(), (mn * r[1]).contiguous()


def _seed_of(seed, k):
    return (seed * 1000003 + k * 7919 + 12345) & 0xFFFFFFFFFFFF


class Saved:
    """A saved tensor as a program keeps it: codes, running estimates, and the position in its random stream."""

    def __init__(self, x, L, g, seed, stochastic=True, op=None, dims=None):
        self.x, self.L, self.seed, self.offset = x, L, seed, 0
        self.alpha, self.beta = _estimates(x, L, g)
        self.q = torch.empty(x.numel(), dtype=torch.int8, device=DEV)
        self.mode = m.ROUND_STOCHASTIC if stochastic else m.ROUND_NEAREST_EVEN
        self.ws = _workspace(m.OP_UPDATE_RUNNING_PARAMS if op is None else op, *(L if dims is None else dims), x.dtype)

    def step(self):
        """the offset of this call; the next call's starts behind the blocks that this one uses"""
        at = self.offset
        self.offset += -(-self.q.numel() // 8)
        return at

    def forward(self):
        m.mesa_update_running_params(self.x, self.L, self.alpha, self.beta, LAM, False, self.ws)
        m.mesa_quantize_headwise(self.x, self.L, self.alpha, self.beta, self.q, self.mode, self.seed, self.step())


def _workspace(op, a, b, c, dt):
    return torch.empty(max(16, m.workspace_bytes(op, a, b, c, MESA_DTYPES[dt])), dtype=torch.uint8, device=DEV)


def _codes(x, L, g):
    """Codes of x that an earlier forward left behind (nearest rounding), with the estimates they were taken with."""
    alpha, beta = _estimates(x, L, g)
    return _plain_codes(x, L, alpha, beta, None), alpha, beta


def prepare(case, seed):
    return {"saved": _prep_saved, "softmax": _prep_softmax, "gelu": _prep_gelu, "layernorm": _prep_layernorm, "linear": _prep_linear,
            "attention": _prep_attention, "conv": _prep_conv, "block": _prep_block}[case["kind"]](case, seed)


def _inputs_saved(c, seed):
    """x of the case: an attention map where a group is a square, else activations"""
    g, dt, L = _gen(seed), DTYPES[c["dtype"]], (c["outer"], c["groups"], c["inner"])
    N = math.isqrt(L[2])
    if N * N == L[2] and N > 16:
        return _map(L[0], L[1], N, g, dt), L, g
    return _tokens((L[0], L[1] * L[2]), g, dt), L, g


def _prep_saved(c, seed):
    x, L, g = _inputs_saved(c, seed)
    s = Saved(x, L, g, _seed_of(seed, 1), c["stochastic"])
    return dict(case=c, s=s, x_hat=torch.empty_like(x))


def _prep_softmax(c, seed):
    g, dt, B, H, N = _gen(seed), DTYPES[c["dtype"]], c["B"], c["H"], c["N"]
    logits = _logits(B, H, N, g, dt)
    s = Saved(torch.softmax(logits[:1].float(), -1).to(dt), (1, H, N * N), g, _seed_of(seed, 2), c["stochastic"], m.OP_SOFTMAX_FWD_Q,
              (B * H * N, H, N))
    s.q = torch.empty(logits.numel(), dtype=torch.int8, device=DEV)
    s.x = logits
    dy = _normal(logits.shape, g, dt)
    old = _codes(_map(B, H, N, g, dt), (B, H, N * N), g)
    return dict(case=c, s=s, y=torch.empty_like(logits), old=old, dy=dy, dx=torch.empty_like(dy))


def _prep_gelu(c, seed):
    g, dt, M, D, G = _gen(seed), DTYPES[c["dtype"]], c["M"], c["D"], c["G"]
    x = _normal((M, D), g, dt)
    s = Saved(x, (M, G, D // G), g, _seed_of(seed, 3), c["stochastic"])
    dy = _normal((M, D), g, dt)
    old = _codes(_normal((M, D), g, dt), s.L, g)
    return dict(case=c, s=s, y=torch.empty_like(x), old=old, dy=dy, dx=torch.empty_like(dy))


def _prep_layernorm(c, seed):
    g, dt, M, D, G = _gen(seed), DTYPES[c["dtype"]], c["M"], c["D"], c["G"]
    x = _tokens((M, D), g, dt)
    s = Saved(x, (M, G, D // G), g, _seed_of(seed, 4), c["stochastic"], m.OP_LAYERNORM_FWD_Q, (M, D, G))
    st = dict(case=c, s=s, y=torch.empty_like(x), mean=torch.empty(M, device=DEV), rstd=torch.empty(M, device=DEV))
    st["bias"] = (0.1 * _normal((D,), g)).to(dt)
    old = _tokens((M, D), g, dt)
    st["old"], st["old_stats"] = _codes(old, s.L, g), _ln_stats(old)
    st.update(_ln_backward(M, D, G, g, dt))
    return st


def _ln_stats(x):
    x = x.float()
    return x.mean(-1).contiguous(), torch.rsqrt(x.var(-1, unbiased=False) + EPS).contiguous()


def _ln_backward(M, D, G, g, dt):
    gamma = (0.5 + torch.rand(D, generator=g, device=DEV)).to(dt)
    dy = _normal((M, D), g, dt)
    return dict(gamma=gamma, dy=dy, dx=torch.empty_like(dy), dgamma=torch.empty(D, device=DEV), dbeta=torch.empty(D, device=DEV),
                ws=_workspace(m.OP_LAYERNORM_BWD_Q, M, D, G, dt))


def _prep_linear(c, seed):
    g, dt, M, K, G, N = _gen(seed), DTYPES[c["dtype"]], c["M"], c["K"], c["G"], c["N_out"]
    xq, alpha, beta = _codes(_tokens((M, K), g, dt), (M, G, K // G), g)
    return dict(case=c, xq=xq, alpha=alpha, beta=beta, **_linear_backward(M, K, N, g, dt))


def _linear_backward(M, K, N, g, dt):
    dy = _normal((M, N), g, dt)
    return dict(dy=dy, dW=torch.empty((N, K), device=DEV), db=torch.empty(N, device=DEV), ws=_workspace(m.OP_LINEAR_DW_Q, M, K, N, dt))


def _prep_attention(c, seed):
    g, dt, B, H, N, Dh = _gen(seed), DTYPES[c["dtype"]], c["B"], c["H"], c["N"], c["Dh"]
    st = dict(case=c, scale=Dh ** -0.5)
    for name in "qkv":
        st[name] = _codes(_normal((B, H, N, Dh), g, dt), (B, H, N * Dh), g)
    st["a"] = _codes(_map(B, H, N, g, dt), (B, H, N * N), g)
    st.update(_attention_backward(B, H, N, Dh, g, dt))
    return st


def _attention_backward(B, H, N, Dh, g, dt):
    dO = _normal((B, H, N, Dh), g, dt)
    return dict(dO=dO, dA=torch.empty((B, H, N, N), dtype=dt, device=DEV), dS=torch.empty((B, H, N, N), dtype=dt, device=DEV), dQ=torch.empty_like(dO),
                dK=torch.empty_like(dO), dV=torch.empty_like(dO))


def _conv2d(c):
    p = c["k"] // 2
    return m.Conv2d(c["B"], c["C_in"], c["H"], c["W"], c["C_out"], c["k"], c["k"], 1, 1, p, p, 1, 1)


def _prep_conv(c, seed):
    g, dt = _gen(seed), DTYPES[c["dtype"]]
    B, C, H, W, G = c["B"], c["C_in"], c["H"], c["W"], c["G"]
    cv = _conv2d(c)
    x = torch.relu(_normal((B, C, H, W), g, dt))
    xq, alpha, beta = _codes(x, (B, G, C // G * H * W), g)
    dy = _normal((B, c["C_out"], *cv.out_hw()), g, dt)
    n = m.conv2d_dw_q_workspace_bytes(cv, MESA_DTYPES[dt])
    return dict(case=c, cv=cv, xq=xq, alpha=alpha, beta=beta, dy=dy, dW=torch.empty((c["C_out"], C, c["k"], c["k"]), device=DEV),
                db=torch.empty(c["C_out"], device=DEV), ws=torch.empty(max(16, n), dtype=torch.uint8, device=DEV))


BLOCK_TENSORS = ("ln1", "qkv", "q", "k", "v", "a", "proj", "ln2", "fc1", "gelu", "fc2")


def _block_dims(c):
    """name -> (layout) of a block's saved tensors"""
    B, N, D, H, F = c["B"], c["N"], c["D"], c["H"], c["mlp"]
    tok, head, wide = (B * N, H, D // H), (B, H, N * (D // H)), (B * N, H, F // H)
    return dict(ln1=tok, qkv=tok, q=head, k=head, v=head, a=(B, H, N * N), proj=tok, ln2=tok, fc1=tok, gelu=wide, fc2=wide)


def _prep_block(c, seed):
    g, dt, B, N, D, H, F = _gen(seed), DTYPES[c["dtype"]], c["B"], c["N"], c["D"], c["H"], c["mlp"]
    st, saved = dict(case=c), {}
    for k, (name, L) in enumerate(_block_dims(c).items()):
        if name == "a":
            x = _map(B, H, N, g, dt)
        elif name in ("q", "k", "v", "gelu"):
            x = _normal((L[0], L[1] * L[2]), g, dt)
        elif name == "fc2":
            x = torch.nn.functional.gelu(_normal((L[0], L[1] * L[2]), g, dt))
        else:
            x = _tokens((L[0], L[1] * L[2]), g, dt)
        saved[name] = Saved(x, L, g, _seed_of(seed, 10 + k), c["stochastic"])
    st["saved"] = saved
    for name, (K, n) in dict(qkv=(D, 3 * D), proj=(D, D), fc1=(D, F), fc2=(F, D)).items():
        st["d" + name] = _linear_backward(B * N, K, n, g, dt)
    for name in ("ln1", "ln2"):
        st["d" + name] = _ln_backward(B * N, D, H, g, dt)
        st["d" + name]["mean"], st["d" + name]["rstd"] = _ln_stats(saved[name].x)
    st["dgelu"] = dict(dy=_normal((B * N, F), g, dt), dx=torch.empty((B * N, F), dtype=dt, device=DEV))
    st["dattn"] = _attention_backward(B, H, N, D // H, g, dt)
    st["scale"] = (D // H) ** -0.5
    return st


# -------------------------------------------------------------------------------------------------------------- one pass
def run(st):
    return {"saved": _run_saved, "softmax": _run_softmax, "gelu": _run_gelu, "layernorm": _run_layernorm, "linear": _run_linear,
            "attention": _run_attention, "conv": _run_conv, "block": _run_block}[st["case"]["kind"]](st)


def _run_saved(st):
    s = st["s"]
    s.forward()
    m.mesa_dequantize(s.q, s.L, s.alpha, s.beta, st["x_hat"])
    return dict(q=s.q, alpha=s.alpha, beta=s.beta, x_hat=st["x_hat"])


def _run_softmax(st):
    c, s = st["case"], st["s"]
    B, H, N = c["B"], c["H"], c["N"]
    m.mesa_softmax_fwd_q(s.x, B, H, N, N, s.alpha, s.beta, LAM, st["y"], s.q, s.ws, s.mode, s.seed, s.step())
    m.mesa_softmax_bwd_q(st["old"][0], B, H, N, N, st["old"][1], st["old"][2], st["dy"], st["dx"])
    return dict(y=st["y"], q=s.q, alpha=s.alpha, beta=s.beta, dx=st["dx"])


def _run_gelu(st):
    s = st["s"]
    m.mesa_gelu_fwd_q(s.x, s.L, s.alpha, s.beta, LAM, st["y"], s.q, s.ws, s.mode, s.seed, s.step())
    m.mesa_gelu_bwd_q(st["old"][0], s.L, st["old"][1], st["old"][2], st["dy"], st["dx"])
    return dict(y=st["y"], q=s.q, alpha=s.alpha, beta=s.beta, dx=st["dx"])


def _run_layernorm(st):
    c, s = st["case"], st["s"]
    M, D, G = c["M"], c["D"], c["G"]
    m.mesa_layernorm_fwd_q(s.x, M, D, G, st["gamma"], st["bias"], EPS, s.alpha, s.beta, LAM, st["y"], st["mean"], st["rstd"], s.q, s.ws,
                           s.mode, s.seed, s.step())
    m.mesa_layernorm_bwd_q(st["old"][0], M, D, G, st["old"][1], st["old"][2], *st["old_stats"], st["gamma"], st["dy"], st["dx"], st["dgamma"],
                           st["dbeta"], st["ws"])
    return dict(y=st["y"], mean=st["mean"], rstd=st["rstd"], q=s.q, alpha=s.alpha, beta=s.beta, dx=st["dx"], dgamma=st["dgamma"], dbeta=st["dbeta"])


def _run_linear(st):
    c = st["case"]
    m.mesa_linear_dw_q(st["xq"], c["M"], c["K"], c["G"], st["alpha"], st["beta"], st["dy"], c["N_out"], st["dW"], st["db"], st["ws"])
    return dict(dW=st["dW"], db=st["db"])


def _attention(dims, q, k, v, a, d, scale):
    B, H, N, Dh = dims
    m.mesa_attn_av_bwd_q(a[0], v[0], B, H, N, Dh, a[1], a[2], v[1], v[2], d["dO"], d["dA"], d["dV"])
    m.mesa_softmax_bwd_q(a[0], B, H, N, N, a[1], a[2], d["dA"], d["dS"])
    m.mesa_attn_qk_bwd_q(q[0], k[0], B, H, N, Dh, q[1], q[2], k[1], k[2], d["dS"], scale, d["dQ"], d["dK"])
    return dict(dA=d["dA"], dS=d["dS"], dQ=d["dQ"], dK=d["dK"], dV=d["dV"])


def _run_attention(st):
    c = st["case"]
    return _attention((c["B"], c["H"], c["N"], c["Dh"]), st["q"], st["k"], st["v"], st["a"], st, st["scale"])


def _run_conv(st):
    m.mesa_conv2d_dw_q(st["xq"], st["cv"], st["case"]["G"], st["alpha"], st["beta"], st["dy"], st["dW"], st["db"], st["ws"])
    return dict(dW=st["dW"], db=st["db"])


def _run_block(st):
    c, saved = st["case"], st["saved"]
    B, N, D, H, F = c["B"], c["N"], c["D"], c["H"], c["mlp"]
    for name in BLOCK_TENSORS:
        saved[name].forward()
    out = {name: dict(q=s.q, alpha=s.alpha, beta=s.beta) for name, s in saved.items()}

    def linear(name, K, n):
        s, d = saved[name], st["d" + name]
        m.mesa_linear_dw_q(s.q, B * N, K, H, s.alpha, s.beta, d["dy"], n, d["dW"], d["db"], d["ws"])
        out["d" + name] = dict(dW=d["dW"], db=d["db"])

    def layernorm(name):
        s, d = saved[name], st["d" + name]
        m.mesa_layernorm_bwd_q(s.q, B * N, D, H, s.alpha, s.beta, d["mean"], d["rstd"], d["gamma"], d["dy"], d["dx"], d["dgamma"], d["dbeta"], d["ws"])
        out["d" + name] = dict(dx=d["dx"], dgamma=d["dgamma"], dbeta=d["dbeta"])

    linear("fc2", F, D)
    s, d = saved["gelu"], st["dgelu"]
    m.mesa_gelu_bwd_q(s.q, s.L, s.alpha, s.beta, d["dy"], d["dx"])
    out["dgelu"] = d["dx"]
    linear("fc1", D, F)
    layernorm("ln2")
    linear("proj", D, D)
    q, k, v, a = ((saved[n].q, saved[n].alpha, saved[n].beta) for n in "qkva")
    out["dattn"] = _attention((B, H, N, D // H), q, k, v, a, st["dattn"], st["scale"])
    linear("qkv", D, 3 * D)
    layernorm("ln1")
    return out


# ------------------------------------------------------------------------------------------------------ what a pass needs
def work(case):
    """Bytes and operations that one pass cannot do without: what a call is given is read once, what it returns is written once."""
    c, e = case, {"f16": 2, "bf16": 2, "f32": 4}[case["dtype"]]
    kind = c["kind"]
    if kind == "saved":
        n = c["outer"] * c["groups"] * c["inner"]
        return dict(bytes=n * (e + 1) + n * (1 + e), flops=0)
    if kind == "softmax":
        n = c["B"] * c["H"] * c["N"] ** 2
        return dict(bytes=n * (2 * e + 1) + n * (1 + 2 * e), flops=0)
    if kind in ("gelu", "layernorm"):
        n, rows = c["M"] * c["D"], (c["M"] if kind == "layernorm" else 0)
        return dict(bytes=n * (2 * e + 1) + n * (1 + 2 * e) + rows * 16, flops=0)
    if kind == "linear":
        return _work_linear(c["M"], c["K"], c["N_out"], e)
    if kind == "attention":
        return _work_attention(c["B"] * c["H"], c["N"], c["Dh"], e)
    if kind == "conv":
        hw, kk = c["H"] * c["W"], c["k"] * c["k"]
        return dict(bytes=c["B"] * hw * (c["C_in"] + e * c["C_out"]) + 4 * c["C_in"] * c["C_out"] * kk, flops=2 * c["B"] * hw * c["C_in"] * c["C_out"] * kk)
    B, N, D, H, F = c["B"], c["N"], c["D"], c["H"], c["mlp"]
    n = sum(L[0] * L[1] * L[2] for L in _block_dims(c).values())
    parts = [dict(bytes=n * (e + 1), flops=0), dict(bytes=B * N * F * (1 + 2 * e), flops=0), dict(bytes=2 * B * N * (D * (1 + 2 * e) + 8), flops=0),
             _work_attention(B * H, N, D // H, e)]
    parts += [_work_linear(B * N, K, o, e) for K, o in ((D, 3 * D), (D, D), (D, F), (F, D))]
    return {k: sum(p[k] for p in parts) for k in ("bytes", "flops")}


def _work_linear(M, K, N, e):
    return dict(bytes=M * K + e * M * N + 4 * N * K, flops=2 * M * N * K)


def _work_attention(heads, N, Dh, e):
    """dA written and read by softmax's backward, dS written and read by the Q K^T product; codes of A read by both calls that take them"""
    return dict(bytes=heads * (N * N * (2 + 4 * e) + N * Dh * (3 + 4 * e)), flops=8 * heads * N * N * Dh)


#: Largest relative error, largest single difference and share of codes that may differ, by storage type: four times what a pass
#: is off its results in 64 bits (binary16 3.6e-4 and bfloat16 2.9e-3 where three roundings to the storage type follow each other,
#: binary32 4e-6 in the weight gradients); a softmax summed in another order rounds one stored probability in some thousands to
#: its neighbour, which moves fewer than one code in a million.
TOLERANCE = {
    "f16": dict(rel=1.5e-3, max=2e-2, differ=1e-5),
    "bf16": dict(rel=1.2e-2, max=1e-1, differ=1e-5),
    "f32": dict(rel=1.5e-5, max=5e-4, differ=1e-5),
}


def tolerance(case):
    if case["kind"] == "saved":
        return "exact"
    return dict(TOLERANCE[case["dtype"]])


# ------------------------------------------------------------------------------------------------------- the same in 64 bits
def _philox(seed, offset, blocks):
    """Philox-4x32-10 (Salmon et al., 2011), counter words 0 and 1 = offset + block, key = seed: (blocks, 4) words"""
    low = 0xFFFFFFFF
    n = torch.arange(offset, offset + blocks, dtype=torch.int64, device=DEV)
    c = [n & low, (n >> 32) & low, torch.zeros_like(n), torch.zeros_like(n)]
    k0, k1 = seed & low, (seed >> 32) & low
    for _ in range(10):
        p0, p1 = c[0] * 0xD2511F53, c[2] * 0xCD9E8D57         # the low 64 bits; hi and lo halves below
        c = [((p1 >> 32) & low) ^ c[1] ^ k0, p1 & low, ((p0 >> 32) & low) ^ c[3] ^ k1, p0 & low]
        k0, k1 = (k0 + 0x9E3779B9) & low, (k1 + 0xBB67AE85) & low
    return torch.stack(c, dim=1)


def _fractions(seed, offset, numel):
    """the uniform numbers of elements 0 .. numel-1: 16 bits each, two to a word, the low half first"""
    w = _philox(seed, offset, -(-numel // 8))
    bits = torch.stack([w & 0xFFFF, w >> 16], dim=2).reshape(-1)[:numel]
    return bits.float() * 2.0 ** -16


def _plain_codes(x, L, alpha, beta, u):
    """Codes as they are defined: binary32, each operation rounded; u None: nearest, ties to even"""
    a = alpha.cpu()
    r = torch.where(a > 0, torch.full_like(a, 255) / a, torch.zeros_like(a)).to(DEV).view(1, -1, 1)
    q = torch.empty(x.numel(), dtype=torch.int8, device=DEV)
    per = max(1, (1 << 27) // (L[1] * L[2]))
    for at in range(0, L[0], per):
        end = min(L[0], at + per)
        lo, hi = at * L[1] * L[2], end * L[1] * L[2]
        v = (x.view(-1)[lo:hi].float().view(end - at, L[1], L[2]) - beta.view(1, -1, 1)) * r
        v = torch.round(v) if u is None else torch.floor(v + u[lo:hi].view_as(v))
        q[lo:hi] = (v.clamp(0, 255) - 128).to(torch.int8).view(-1)
    return q


def _plain_estimates(x, L, alpha, beta):
    """the running estimates moved by the extrema of x, binary32 with every operation rounded"""
    v = x.view(L)
    mn, mx = v.amin(dim=(0, 2)).float().cpu(), v.amax(dim=(0, 2)).float().cpu()
    lam = torch.tensor(LAM, dtype=torch.float32)
    a, b = alpha.cpu(), beta.cpu()
    return (lam * a + (1 - lam) * (mx - mn)).to(DEV), (lam * b + (1 - lam) * mn).to(DEV)


def _x_hat(q, L, alpha, beta):
    a, b = alpha.double().view(1, -1, 1), beta.double().view(1, -1, 1)
    return (q.view(L).double() + 128) * (a / 255) + b


def _exact_saved(s):
    """two-call forward: (codes, alpha, beta)"""
    a, b = _plain_estimates(s.x, s.L, s.alpha, s.beta)
    u = _fractions(s.seed, 0, s.x.numel()) if s.mode == m.ROUND_STOCHASTIC else None
    return _plain_codes(s.x, s.L, a, b, u), a, b


def _gelu_grad(x):
    return 0.5 * (1 + torch.erf(x * math.sqrt(0.5))) + x * torch.exp(-0.5 * x * x) / math.sqrt(2 * math.pi)


def _exact_softmax_bwd(y_hat, dy):
    return y_hat * (dy - (dy * y_hat).sum(-1, keepdim=True))


def _exact_layernorm_bwd(x_hat, mean, rstd, gamma, dy):
    xn = (x_hat - mean.double().view(-1, 1)) * rstd.double().view(-1, 1)
    gd = dy * gamma.double()
    dx = rstd.double().view(-1, 1) * (gd - gd.mean(-1, keepdim=True) - xn * (gd * xn).mean(-1, keepdim=True))
    return dict(dx=dx, dgamma=(dy * xn).sum(0), dbeta=dy.sum(0))


def _exact_linear(x_hat, dy):
    dy = dy.double()
    return dict(dW=dy.t().contiguous() @ x_hat, db=dy.sum(0))


def _exact_attention(dims, q, k, v, a, dO, scale):
    B, H, N, Dh = dims
    hat = lambda t, inner: _x_hat(t[0], (B, H, inner), t[1], t[2]).view(B * H, N, -1)  # noqa: E731
    dO = dO.double().view(B * H, N, Dh)
    V, A = hat(v, N * Dh), hat(a, N * N)
    dA = torch.bmm(dO, V.transpose(1, 2).contiguous())
    dV = torch.bmm(A.transpose(1, 2).contiguous(), dO)
    dS = _exact_softmax_bwd(A, dA)
    del A, V
    dQ = scale * torch.bmm(dS, hat(k, N * Dh))
    dK = scale * torch.bmm(dS.transpose(1, 2).contiguous(), hat(q, N * Dh))
    return dict(dA=dA.view(B, H, N, N), dS=dS.view(B, H, N, N), dQ=dQ.view(B, H, N, Dh), dK=dK.view(B, H, N, Dh), dV=dV.view(B, H, N, Dh))


def exact(case, seed):
    c, st, kind = case, prepare(case, seed), case["kind"]
    if kind == "saved":
        q, a, b = _exact_saved(st["s"])
        return dict(q=None, alpha=a.double(), beta=b.double(), x_hat=_x_hat(q, st["s"].L, a, b).view(st["s"].x.shape))
    if kind == "softmax":
        s, B, H, N = st["s"], c["B"], c["H"], c["N"]
        y = torch.softmax(s.x.double(), -1)
        a, b = _plain_estimates(y.to(s.x.dtype), (B, H, N * N), s.alpha, s.beta)
        dx = _exact_softmax_bwd(_x_hat(st["old"][0], (B, H, N * N), *st["old"][1:]).view(B, H, N, N), st["dy"].double())
        return dict(y=y, q=None, alpha=a.double(), beta=b.double(), dx=dx)
    if kind == "gelu":
        s = st["s"]
        a, b = _plain_estimates(s.x, s.L, s.alpha, s.beta)
        dx = _gelu_grad(_x_hat(st["old"][0], s.L, *st["old"][1:]).view(s.x.shape)) * st["dy"].double()
        x = s.x.double()
        return dict(y=0.5 * x * (1 + torch.erf(x * math.sqrt(0.5))), q=None, alpha=a.double(), beta=b.double(), dx=dx)
    if kind == "layernorm":
        s = st["s"]
        a, b = _plain_estimates(s.x, s.L, s.alpha, s.beta)
        x = s.x.double()
        mean, var = x.mean(-1), x.var(-1, unbiased=False)
        rstd = torch.rsqrt(var + EPS)
        y = (x - mean.view(-1, 1)) * rstd.view(-1, 1) * st["gamma"].double() + st["bias"].double()
        back = _exact_layernorm_bwd(_x_hat(st["old"][0], s.L, *st["old"][1:]).view(x.shape), *st["old_stats"], st["gamma"], st["dy"].double())
        return dict(y=y, mean=mean, rstd=rstd, q=None, alpha=a.double(), beta=b.double(), **back)
    if kind == "linear":
        M, K, G = c["M"], c["K"], c["G"]
        return _exact_linear(_x_hat(st["xq"], (M, G, K // G), st["alpha"], st["beta"]).view(M, K), st["dy"])
    if kind == "attention":
        return _exact_attention((c["B"], c["H"], c["N"], c["Dh"]), st["q"], st["k"], st["v"], st["a"], st["dO"], st["scale"])
    if kind == "conv":
        B, C, H, W, k = c["B"], c["C_in"], c["H"], c["W"], c["k"]
        p = k // 2
        x = torch.nn.functional.pad(_x_hat(st["xq"], (B, c["G"], C // c["G"] * H * W), st["alpha"], st["beta"]).view(B, C, H, W), (p, p, p, p))
        dy = st["dy"].double().transpose(0, 1).reshape(c["C_out"], -1)
        dW = torch.stack([dy @ x[:, :, i:i + H, j:j + W].permute(0, 2, 3, 1).reshape(-1, C) for i in range(k) for j in range(k)], -1)
        return dict(dW=dW.view(c["C_out"], C, k, k), db=dy.sum(1))
    B, N, D, H, F = c["B"], c["N"], c["D"], c["H"], c["mlp"]
    out, codes = {}, {}
    for name, s in st["saved"].items():
        codes[name] = _exact_saved(s)
        out[name] = dict(q=None, alpha=codes[name][1].double(), beta=codes[name][2].double())
    hat = lambda name: _x_hat(codes[name][0], st["saved"][name].L, *codes[name][1:]).view(B * N, -1)  # noqa: E731
    for name in ("qkv", "proj", "fc1", "fc2"):
        out["d" + name] = _exact_linear(hat(name), st["d" + name]["dy"])
    for name in ("ln1", "ln2"):
        d = st["d" + name]
        out["d" + name] = _exact_layernorm_bwd(hat(name), d["mean"], d["rstd"], d["gamma"], d["dy"].double())
    out["dgelu"] = _gelu_grad(hat("gelu")) * st["dgelu"]["dy"].double()
    out["dattn"] = _exact_attention((B, H, N, D // H), codes["q"], codes["k"], codes["v"], codes["a"], st["dattn"]["dO"], st["scale"])
    return out
