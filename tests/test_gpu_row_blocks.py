"""LayerNorm forward and backward where a workgroup walks several blocks of rows: one, two, three and four of them, the last
one whole, short by a row, or a row and nothing more; rows that fill their lanes and rows that leave some idle.  The kernels
leave lanes without an element to the hardware's bounds check, so the outputs lie between sentinels.

Bounds: those of the other tests of these layers; codes, running estimates and sentinels bit for bit.
"""
import numpy as np
import pytest
import torch

from oracle import mesa_ref as R
from tests.test_gpu_parity import DTYPE_IDS, DTYPES, TOL, M, canon, npy, relerr, ws_for  # noqa: F401

pytestmark = pytest.mark.gpu

# rows of a round of workgroups (backward / forward): 65536 / 49152 at 8 columns, 16384 / 24576 at 192 and / 12288 at 256, 8192 / 12288 at 384 and / 6144 at 512,
# 4096 / 6144 at 768 and 1024 (forward in binary32 3072 at 1024), - / 3072 at 1280, - / 2048 beyond 1536.  Below a round the forward of rows that come one per lane
# group and block (three and four vectors per lane, two in binary32) has two blocks per workgroup already.
SHAPES = [(65537, 8, 1), (98303, 8, 1), (16385, 192, 3), (12287, 256, 4), (24577, 192, 3), (49153, 192, 3), (73729, 192, 3), (8193, 384, 6), (24593, 384, 6), (36865, 384, 6), (12289, 512, 8),
          (16383, 384, 6), (4097, 768, 12), (12291, 768, 12), (18433, 768, 12), (6143, 768, 12), (8195, 1024, 16), (9219, 1024, 16), (3073, 1280, 5), (6145, 1280, 5), (9217, 1280, 5), (1025, 2048, 8),
          (4099, 2048, 8), (4097, 1600, 5), (6145, 1544, 1)]


def between(t, fill=3.0):
    """(a tensor like t between sentinels, its middle)"""
    out = torch.full((t.numel() + 256,), fill, dtype=t.dtype, device="cuda")
    return out, out[128:128 + t.numel()].view(t.shape)


def untouched(out, fill=3.0):
    return bool((out[:128] == fill).all()) and bool((out[-128:] == fill).all())


@pytest.mark.parametrize("dtype", DTYPES, ids=DTYPE_IDS)
@pytest.mark.parametrize("rows,D,G", SHAPES)
def test_layernorm_blocks(M, rows, D, G, dtype):  # noqa: F811
    g = torch.Generator(device="cuda").manual_seed(rows + D)
    a, b = torch.full((G,), 9.0, device="cuda"), torch.full((G,), -4.5, device="cuda")
    ra, rb = npy(a).copy(), npy(b).copy()
    gamma = (1 + 0.1 * torch.randn(D, generator=g, device="cuda")).to(dtype)
    bias = (0.1 * torch.randn(D, generator=g, device="cuda")).to(dtype)
    x = (torch.randn((rows, D), generator=g, device="cuda") + 0.3).to(dtype)
    (yo, y), (qo, q) = between(x), between(torch.empty(rows * D, dtype=torch.int8))
    (mo, mean), (so, rstd) = between(torch.empty(rows)), between(torch.empty(rows))
    M.mesa_layernorm_fwd_q(x, rows, D, G, gamma, bias, 1e-5, a, b, 0.9, y, mean, rstd, q, ws_for(M, M.OP_LAYERNORM_FWD_Q, rows, D, G, dtype),
                           M.ROUND_STOCHASTIC, 13, 5)
    assert all(untouched(t) for t in (yo, qo, mo, so))
    ry, rmean, rrstd = R.layernorm_fwd(npy(x), rows, D, npy(gamma), npy(bias), 1e-5)
    assert relerr(npy(y), ry) <= TOL[dtype]
    assert relerr(npy(mean), rmean) <= 1e-5 and relerr(npy(rstd), rrstd) <= 1e-5
    qa, qb = ra, rb
    rq, ra, rb = R.quantize_update_fused(npy(x), (rows, G, D // G), ra, rb, 0.9, R.ROUND_STOCHASTIC, 13, 5)
    assert np.array_equal(npy(q), rq.reshape(-1))
    assert np.array_equal(canon(npy(a)), canon(ra)) and np.array_equal(canon(npy(b)), canon(rb))
    if D > 1024:                                    # the backward's rows in a wave end there
        return
    dy = torch.randn((rows, D), generator=g, device="cuda").to(dtype)
    xo, dx = between(dy)
    dg, db = torch.empty(D, device="cuda"), torch.empty(D, device="cuda")
    old = [torch.from_numpy(t).cuda() for t in (qa, qb)]
    M.mesa_layernorm_bwd_q(q, rows, D, G, *old, mean, rstd, gamma, dy, dx, dg, db, ws_for(M, M.OP_LAYERNORM_BWD_Q, rows, D, G, dtype))
    rdx, rdg, rdb = R.layernorm_bwd_q(npy(q), rows, D, G, qa, qb, npy(mean), npy(rstd), npy(gamma), npy(dy))
    assert untouched(xo) and relerr(npy(dx), rdx) <= TOL[dtype]
    assert relerr(npy(dg), rdg) <= 1e-4 and relerr(npy(db), rdb) <= 1e-4   # binary32 sums of up to 98303 rows
    M.mesa_layernorm_bwd_q(q, rows, D, G, *old, mean, rstd, gamma, dy, dy, dg, db, ws_for(M, M.OP_LAYERNORM_BWD_Q, rows, D, G, dtype))   # in place
    assert torch.equal(dy, dx)
