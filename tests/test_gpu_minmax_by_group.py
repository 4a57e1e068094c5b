"""The running estimates' scan by group: groups of one workgroup and of several, slabs that start anywhere, the ends of the ranges
it is taken for, against the CPU oracle bit for bit."""
import numpy as np
import pytest
import torch

from oracle import mesa_ref as R
from tests.test_gpu_parity import DTYPE_IDS, DTYPES, _mid_of_frame, npy, ws_for

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def M():
    import paper_2111_11124_amd as m
    assert torch.cuda.is_available(), "these tests need the MI355X"
    m.lib()
    return m


@pytest.mark.parametrize("dtype", DTYPES, ids=DTYPE_IDS)
@pytest.mark.parametrize("layout", [(1, 1, 1), (1, 3, 7), (3, 2, 9), (512, 2, 64), (513, 2, 64), (4096, 3, 8), (1, 2, 32767), (1, 2, 32769), (600, 8, 65),
                                    (700, 3, 63), (300, 9, 441), (31, 5, 2047), (40, 3, 2049), (2, 8192, 71), (5000, 2, 341)])
def test_running_estimates_scan_by_group(M, layout, dtype):
    outer, groups, inner = layout
    n = outer * groups * inner
    g = torch.Generator(device="cuda").manual_seed(n)
    a, b = torch.full((groups,), 3.0, device="cuda"), torch.full((groups,), -1.0, device="cuda")
    ra, rb = npy(a).copy(), npy(b).copy()
    ws = ws_for(M, M.OP_UPDATE_RUNNING_PARAMS, *layout, dt=dtype)
    for t in range(3):
        x = torch.randn((outer, groups, inner), device="cuda", generator=g) * (1 + t) + torch.linspace(-2, 2, groups, device="cuda").view(1, -1, 1)
        x = _mid_of_frame(x.to(dtype), 3e4)                 # what lies outside is larger than anything inside
        M.mesa_update_running_params(x, layout, a, b, 0.9, t == 0, ws)
        ra, rb = R.update_running_params(npy(x), layout, ra, rb, 0.9, t == 0)
        assert np.array_equal(npy(a) + np.float32(0), ra + np.float32(0)) and np.array_equal(npy(b) + np.float32(0), rb + np.float32(0)), t
    s = torch.full((groups,), 3.0, device="cuda")
    M.mesa_update_running_scale_sym(x, layout, s, 0.9, False, ws)
    rs = R.update_running_scale_sym(npy(x), layout, np.full(groups, 3.0, np.float32), 0.9, False)
    assert np.array_equal(npy(s), rs)


@pytest.mark.parametrize("dtype", DTYPES, ids=DTYPE_IDS)
@pytest.mark.parametrize("layout", [(32768, 1, 1), (5000, 1, 7), (1023, 2, 1), (1024, 2, 1), (4096, 3, 1), (2047, 1, 9), (819, 2, 31), (1025, 2, 17), (1, 513, 64),
                                    (64, 513, 64), (7, 513, 73), (8, 513, 73), (40, 1000, 900)])
def test_running_estimates_on_either_side_of_the_scans_lines(M, layout, dtype):
    test_running_estimates_scan_by_group(M, layout, dtype)
