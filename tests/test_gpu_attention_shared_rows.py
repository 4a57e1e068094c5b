"""Attention products of one or two heads, every head size, against the CPU oracle (the bounds of the other attention tests): the waves of a workgroup share out the
contraction (k_bmm_waves), whose blocks they do and do not divide.  Kernels whose groups of waves share rows or stages take more heads: test_gpu_attention_kernels.py."""
import pytest
import torch

from tests.test_gpu_parity import _attention_case

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def M():
    import paper_2111_11124_amd as m
    assert torch.cuda.is_available(), "these tests need the MI355X"
    m.lib()
    return m


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16], ids=["f16", "bf16"])
@pytest.mark.parametrize("B,H,N,Dh", [(1, 1, 64, 64), (1, 2, 80, 32), (1, 1, 272, 64), (1, 1, 336, 128), (1, 1, 1024, 64), (1, 1, 1040, 32), (1, 1, 1072, 64),
                                      (1, 1, 1056, 128)])
def test_attention_products_rows_shared_among_wave_groups(M, B, H, N, Dh, dtype):
    _attention_case(M, B, H, N, Dh, dtype)


@pytest.mark.parametrize("dtype", [torch.float32, torch.float16, torch.bfloat16], ids=["f32", "f16", "bf16"])
@pytest.mark.parametrize("B,H,N,Dh", [(1, 1, 129, 40), (1, 2, 257, 64), (1, 1, 289, 96), (1, 1, 511, 64), (1, 1, 513, 64), (1, 1, 545, 32), (1, 1, 577, 72)])
def test_attention_products_stages_shared_among_wave_groups(M, B, H, N, Dh, dtype):
    """Unaligned rows, head sizes without kernels of their own."""
    _attention_case(M, B, H, N, Dh, dtype)
