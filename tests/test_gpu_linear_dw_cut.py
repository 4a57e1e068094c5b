"""The weight gradient by tiles and slices beyond the matrices that a wave per block of rows takes (more than 2048 rows, or 640 tiles of 32 x 32; a host
test holds that these shapes get there): binary32 in one slice and in several, ragged in every extent, in workspaces of fewer slices than it would take,
infinities, NaN and values that are too large to be cut in one row of tiles, the range of binary32; 16 bits in the workspace there is."""
import numpy as np
import pytest
import torch

from tests.test_gpu_binary32_products import _dw
from tests.test_gpu_binary32_range import EXPONENTS, test_linear_dw_over_the_range_of_binary32 as over_the_range
from tests.test_gpu_linear_dw_plans import test_linear_dw_of_small_matrices_in_the_workspace_there_is as in_the_workspace_there_is

pytestmark = pytest.mark.gpu

# (rows, K, N): slices of several stages; one slice
EDGES = [(2049, 16, 4), (2080, 112, 124), (2081, 128, 128), (2111, 144, 132), (2112, 16, 260), (2113, 272, 12), (4100, 256, 4), (4099, 80, 136), (2500, 192, 576),
         (1, 832, 828), (32, 848, 820), (65, 1040, 644), (129, 656, 1028)]
SPOILT = (2100, 48, 20)
RANGE = [(2100, 48, 44), (2113, 144, 132), (33, 832, 828)]
PLANS = [(2084, 384, 1152, 1, 2124), (2560, 128, 120, 2, 2561), (2049, 384, 384, 6, 2115), (2245, 768, 264, 12, 2311)]   # (.., groups, rows that the workspace is sized for)


@pytest.fixture(scope="module")
def M():
    import paper_2111_11124_amd as m
    assert torch.cuda.is_available(), "these tests need the MI355X"
    m.lib()
    return m


@pytest.mark.parametrize("Mr,K,N", EDGES)
def test_linear_dw_cut_edges(M, Mr, K, N):
    """Per row of dW, since the rows' magnitudes differ by sixty binades; 1e-5 is the binary32 bound of the other tests."""
    dW, db, (rW, rb) = _dw(M, Mr, K, N)
    assert (np.abs(dW - rW).max(1) / np.abs(rW).max(1)).max() <= 1e-5
    assert (np.abs(db - rb) / np.maximum(np.abs(rb), np.abs(rW).max(1))).max() <= 1e-5


@pytest.mark.parametrize("slices", [1, 2, 5])
@pytest.mark.parametrize("Mr,K,N", [(2500, 96, 72), (4099, 80, 136), (2300, 512, 512)])
def test_linear_dw_cut_in_a_workspace_of_fewer_slices(M, Mr, K, N, slices):
    g = torch.Generator(device="cuda").manual_seed(Mr + K)
    q = torch.randint(-128, 128, (Mr, K), dtype=torch.int8, device="cuda", generator=g)
    dy = torch.randn((Mr, N), device="cuda", generator=g)
    a, b = torch.full((1,), 0.7, device="cuda"), torch.full((1,), -0.2, device="cuda")
    n = slices * (N * K + N) * 4 + 16
    assert n < M.workspace_bytes(M.OP_LINEAR_DW_Q, Mr, K, N, M.F32)
    frame = torch.full((n + 256,), 0x55, dtype=torch.uint8, device="cuda")
    dW, db = torch.empty((N, K), device="cuda"), torch.empty(N, device="cuda")
    M.mesa_linear_dw_q(q, Mr, K, 1, a, b, dy, N, dW, db, frame[:n])
    ref = dy.double().t().contiguous() @ ((q.double() + 128) * (a.double() / 255) + b.double())
    assert (dW - ref).abs().max() <= 1e-5 * ref.abs().max()
    assert (db - dy.double().sum(0)).abs().max() <= 1e-5 * dy.double().abs().sum(0).max()
    assert torch.all(frame[n:] == 0x55)                     # nothing behind the workspace


@pytest.mark.parametrize("spoil", [float("inf"), -float("inf"), float("nan"), 3.4e38, 1e-42])
def test_linear_dw_cut_extreme_values_stay_in_their_row(M, spoil):
    """An infinity, a NaN, the largest and a subnormal value of dy: every other row of dW is finite and right."""
    Mr, K, N = SPOILT
    dW, _, (rW, _) = _dw(M, Mr, K, N, spoil=spoil)
    rows = np.arange(N) != N // 2
    assert (np.abs(dW - rW)[rows].max(1) / np.abs(rW)[rows].max(1)).max() <= 1e-5
    if not np.isfinite(spoil):
        assert not np.isfinite(dW[N // 2]).any()
    elif spoil < 1:
        assert np.abs(dW - rW)[N // 2].max() <= 1e-5 * np.abs(rW[N // 2]).max()


@pytest.mark.parametrize("at_nan,at_large", [(0, 1), (1, 0), (0, 2), (3, 1), (2, 3), (5, 4)])
def test_linear_dw_cut_with_a_nan_beside_a_large_value(M, at_nan, at_large):
    """Both in one row of dy, in one thread's vector: the NaN stays in its row of dW and hides the large value from nobody."""
    Mr, K, N = SPOILT
    g = torch.Generator(device="cuda").manual_seed(8 * at_nan + at_large)
    q = torch.randint(-128, 128, (Mr, K), dtype=torch.int8, device="cuda", generator=g)
    dy = torch.randn((Mr, N), device="cuda", generator=g)
    dy[33, at_nan], dy[33, at_large] = float("nan"), 1e33
    a, b = torch.full((1,), 0.7, device="cuda"), torch.full((1,), -0.2, device="cuda")
    ws = torch.empty(M.workspace_bytes(M.OP_LINEAR_DW_Q, Mr, K, N, M.F32), dtype=torch.uint8, device="cuda")
    dW, db = torch.empty((N, K), device="cuda"), torch.empty(N, device="cuda")
    M.mesa_linear_dw_q(q, Mr, K, 1, a, b, dy, N, dW, db, ws)
    ref = dy.double().t().contiguous() @ ((q.double() + 128) * (a.double() / 255) + b.double())
    assert torch.isnan(dW[at_nan]).all() and torch.isnan(db[at_nan])
    rest = torch.arange(N, device="cuda") != at_nan
    assert ((dW - ref)[rest].abs().amax(1) <= 1e-5 * ref[rest].abs().amax(1)).all()


@pytest.mark.parametrize("exponents", [EXPONENTS, [e for e in EXPONENTS if e < 60]], ids=["with-large", "cut"])
@pytest.mark.parametrize("Mr,K,N", RANGE)
def test_linear_dw_cut_over_the_range_of_binary32(M, Mr, K, N, exponents):
    over_the_range(M, Mr, K, N, exponents)


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16], ids=["f16", "bf16"])
@pytest.mark.parametrize("Mr,K,N,G,sized_for", PLANS + [(2084, 384, 1152, 1, None), (2084, 384, 1152, 1, 2084)])
def test_linear_dw_by_tiles_in_the_workspace_there_is(M, Mr, K, N, G, sized_for, dtype):
    in_the_workspace_there_is(M, Mr, K, N, G, sized_for, dtype)
