"""The update on the library's own array, with layouts whose scan would run on more workgroups than it has room for: the estimates of the
workspace form, and of the CPU oracle, bit for bit."""
import numpy as np
import pytest
import torch

from oracle import mesa_ref as R
from tests.test_gpu_parity import npy, ws_for

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def M():
    import paper_2111_11124_amd as m
    assert torch.cuda.is_available(), "these tests need the MI355X"
    m.lib()
    return m


@pytest.mark.parametrize("dtype", [torch.float16, torch.float32], ids=["f16", "f32"])
@pytest.mark.parametrize("layout", [(12, 4096, 64), (37, 1024, 49), (37, 768, 256), (84, 1536, 64), (1321, 128, 49), (209, 768, 96), (26, 2048, 96),
                                    (1589, 384, 20), (54, 3072, 64), (2662, 128, 49), (983, 768, 20), (1, 1024, 9001), (8, 768, 24)])
def test_update_on_the_librarys_array_at_its_room(M, layout, dtype):
    outer, groups, inner = layout
    x = torch.randn((outer, groups, inner), device="cuda", generator=torch.Generator(device="cuda").manual_seed(inner)).to(dtype)
    a, b = torch.full((groups,), 3.0, device="cuda"), torch.full((groups,), -1.0, device="cuda")
    wa, wb = a.clone(), b.clone()
    ra, rb = R.update_running_params(npy(x), layout, npy(a).copy(), npy(b).copy(), 0.9, False)
    M.mesa_update_running_params_static(x, layout, a, b, 0.9, False)
    M.mesa_update_running_params(x, layout, wa, wb, 0.9, False, ws_for(M, M.OP_UPDATE_RUNNING_PARAMS, *layout, dt=dtype))
    assert torch.equal(a, wa) and torch.equal(b, wb)
    assert np.array_equal(npy(a) + np.float32(0), ra + np.float32(0)) and np.array_equal(npy(b) + np.float32(0), rb + np.float32(0))
