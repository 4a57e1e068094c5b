"""Extrema in four tables per workgroup and in one (more than 256 groups), the scan with two and with four vectors per thread, and more
partials than one thread of the second launch takes: the estimates against the CPU oracle bit for bit."""
import numpy as np
import pytest
import torch

from oracle import mesa_ref as R
from tests.test_gpu_parity import DTYPE_IDS, DTYPES, npy, ws_for

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def M():
    import paper_2111_11124_amd as m
    assert torch.cuda.is_available(), "these tests need the MI355X"
    m.lib()
    return m


@pytest.mark.parametrize("dtype", DTYPES, ids=DTYPE_IDS)
@pytest.mark.parametrize("layout", [(3000, 1, 9), (70, 256, 600), (70, 257, 600), (9, 255, 4104), (5001, 7, 64), (1, 1, 1 << 24), (1, 1, (1 << 24) + 8),
                                    (4096, 64, 64), (4097, 64, 64), (2, 1, (1 << 23) + 3)])
def test_extrema_of_either_number_of_tables(M, layout, dtype):
    outer, groups, inner = layout
    x = torch.randn((outer, groups, inner), device="cuda", generator=torch.Generator(device="cuda").manual_seed(inner)).to(dtype)
    a, b = torch.full((groups,), 3.0, device="cuda"), torch.full((groups,), -1.0, device="cuda")
    ra, rb = R.update_running_params(npy(x), layout, npy(a).copy(), npy(b).copy(), 0.9, False)
    M.mesa_update_running_params(x, layout, a, b, 0.9, False, ws_for(M, M.OP_UPDATE_RUNNING_PARAMS, *layout, dt=dtype))
    assert np.array_equal(npy(a) + np.float32(0), ra + np.float32(0)) and np.array_equal(npy(b) + np.float32(0), rb + np.float32(0))
    a, b, q = torch.full((groups,), 3.0, device="cuda"), torch.full((groups,), -1.0, device="cuda"), torch.empty(x.numel(), dtype=torch.int8, device="cuda")
    M.mesa_quantize_update_fused(x, layout, a, b, 0.9, q, ws_for(M, M.OP_UPDATE_RUNNING_PARAMS, *layout, dt=dtype), M.ROUND_NEAREST_EVEN, 1, 0)
    assert np.array_equal(npy(a) + np.float32(0), ra + np.float32(0)) and np.array_equal(npy(b) + np.float32(0), rb + np.float32(0))


@pytest.mark.parametrize("dtype", DTYPES, ids=DTYPE_IDS)
@pytest.mark.parametrize("layout", [(900, 32, 40), (900, 33, 40), (400, 33, 96), (400, 128, 96), (400, 128, 88), (400, 129, 96), (500, 128, 97), (2000, 40, 20), (1, 768, 256), (600, 8, 96), (700, 8, 96)])
def test_extrema_on_either_side_of_the_tables_lines(M, layout, dtype):
    test_extrema_of_either_number_of_tables(M, layout, dtype)
