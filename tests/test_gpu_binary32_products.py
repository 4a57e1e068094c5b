"""Binary32 matrix products at de-quantized operands: the weight gradient of a Linear layer and the backward of the attention
products, on the matrix cores as three bfloat16 parts of the binary32 operand, against the CPU oracle.

Bound: every product of a part and a code is exact in binary32, so the only roundings are those of binary32 sums -- the
binary32 bound of the other tests, 1e-5 of the largest result, holds unchanged.
"""
import numpy as np
import pytest
import torch

import mesa_workloads as W
from oracle import mesa_ref as R
from tests.test_gpu_parity import _attention_case, _mid_of_frame, npy, relerr

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def M():
    import paper_2111_11124_amd as m
    assert torch.cuda.is_available(), "these tests need the MI355X"
    m.lib()
    return m


def _dw(M, Mr, K, N, few=False, spoil=None):
    g = torch.Generator(device="cuda").manual_seed(Mr * 31 + K + N)
    H = 1 if K % 3 else 3
    q = _mid_of_frame(torch.randint(-128, 128, (Mr * K,), dtype=torch.int8, device="cuda", generator=g), 127)
    # magnitudes over sixty binades, so that the parts of a value lie far apart from its neighbours'
    dy = torch.randn((Mr, N), generator=g, device="cuda") * torch.exp2(torch.randint(-30, 31, (1, N), generator=g, device="cuda").float())
    if spoil is not None:
        dy[Mr // 2, N // 2] = spoil
    dy = _mid_of_frame(dy, float("nan"))
    a = 0.5 + torch.rand(H, device="cuda", generator=g)
    b = -torch.rand(H, device="cuda", generator=g)
    n = M.workspace_bytes(M.OP_LINEAR_DW_Q, Mr, K, N, M.F32)
    if few:                                            # one slice: what the call needed at the least
        n = (N * K + N) * 4 + 16
    ws = torch.empty(max(16, n), dtype=torch.uint8, device="cuda")
    dW, db = torch.empty((N, K), device="cuda"), torch.empty(N, device="cuda")
    M.mesa_linear_dw_q(q, Mr, K, H, a, b, dy, N, dW, db, ws)
    return npy(dW).astype(np.float64), npy(db).astype(np.float64), R.linear_dw_q(npy(q), Mr, K, H, npy(a), npy(b), npy(dy), N)


@pytest.mark.parametrize("Mr,K,N", [(1, 16, 4), (31, 112, 124), (32, 128, 128), (33, 144, 132), (63, 16, 260), (64, 256, 4), (65, 272, 12),
                                    (129, 48, 128), (1000, 192, 576), (4099, 80, 136)])
def test_linear_dw_binary32_edges(M, Mr, K, N):
    """Ragged last rows, tiles that end inside, at and behind N and K; per row of dW, since the rows' magnitudes differ by sixty binades.  (All but the
    last are small enough for k_dw_waves; the tiles and slices of k_dw_cut: test_gpu_linear_dw_cut.py.)"""
    dW, db, (rW, rb) = _dw(M, Mr, K, N)
    assert (np.abs(dW - rW).max(1) / np.abs(rW).max(1)).max() <= 1e-5
    # a column sum of dy can cancel; the bound is on its terms' magnitude, which the largest entry of the row carries
    assert (np.abs(db - rb) / np.maximum(np.abs(rb), np.abs(rW).max(1))).max() <= 1e-5


def test_linear_dw_binary32_in_a_workspace_of_one_slice(M):
    dW, db, (rW, rb) = _dw(M, 500, 96, 72, few=True)
    assert (np.abs(dW - rW).max(1) / np.abs(rW).max(1)).max() <= 1e-5


@pytest.mark.parametrize("spoil", [float("inf"), -float("inf"), float("nan"), 3.4e38, 1e-42])
def test_linear_dw_binary32_extreme_values_stay_in_their_row(M, spoil):
    """An infinity, a NaN, the largest and a subnormal value of dy: every other row of dW is finite and right."""
    dW, _, (rW, _) = _dw(M, 70, 48, 20, spoil=spoil)
    rows = np.arange(20) != 10
    assert (np.abs(dW - rW)[rows].max(1) / np.abs(rW)[rows].max(1)).max() <= 1e-5
    if not np.isfinite(spoil):
        assert not np.isfinite(dW[10]).any()
    elif spoil < 1:
        assert np.abs(dW - rW)[10].max() <= 1e-5 * np.abs(rW[10]).max()


@pytest.mark.parametrize("B,H,N,Dh", [(1, 1, 8, 8), (2, 3, 19, 24), (1, 2, 32, 64), (1, 1, 63, 40), (1, 2, 64, 64), (1, 1, 65, 72), (1, 2, 128, 96),
                                      (1, 1, 129, 128), (1, 3, 197, 64), (1, 1, 300, 33)])
def test_attention_products_binary32(M, B, H, N, Dh):
    """Tiles and blocks of steps that end inside, at and behind the extents."""
    _attention_case(M, B, H, N, Dh, torch.float32)


def test_attention_products_binary32_use_nothing_from_outside_their_inputs(M):
    from tests.test_gpu_parity import test_attention_matmul_backward_uses_nothing_from_outside_its_inputs as framed
    for shape in ((1, 2, 49, 32), (1, 1, 100, 33), (1, 1, 197, 64)):
        framed(M, *shape, torch.float32)
