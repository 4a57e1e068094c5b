"""Every kernel of the attention products at least once, in every type: shapes that reach each of them (a host test holds that, for the lines between them move),
against the same products in binary64, and nothing outside an output is written and nothing outside an input reaches a result."""
import pytest
import torch

from tests.test_gpu_attention_waves import run

pytestmark = pytest.mark.gpu

SIXTEEN = [
    # the plain and the general kernel, few heads
    (1, 1, 4, 4), (1, 900, 8, 16), (1, 700, 100, 40), (1, 300, 101, 130), (1, 1, 8, 16), (1, 1, 8, 72), (1, 1, 8, 130), (1, 160, 8, 130), (1, 28, 128, 130), (1, 1, 705, 128), (1, 60, 71, 64),
    # a workgroup per head or per 32 rows
    (1, 900, 8, 32), (1, 450, 33, 32), (1, 200, 71, 32), (1, 900, 8, 64), (1, 900, 33, 64), (1, 400, 72, 64), (1, 640, 8, 96), (1, 300, 63, 96), (1, 257, 72, 96), (1, 640, 8, 128), (1, 640, 33, 128),
    (1, 300, 71, 128), (1, 520, 101, 128), (1, 640, 49, 128),
    # by tiles with one, two and four groups of waves, of aligned rows and of rows that start anywhere
    (1, 257, 80, 32), (1, 130, 128, 32), (1, 130, 131, 32), (1, 513, 131, 32), (1, 20, 1031, 32), (1, 14, 1200, 32), (1, 28, 1040, 32), (1, 450, 64, 64), (1, 513, 131, 64), (1, 160, 197, 64), (1, 160, 208, 64),
    (1, 28, 1024, 64), (1, 28, 1040, 64), (1, 28, 1031, 64), (1, 200, 96, 96), (1, 160, 128, 96), (1, 160, 131, 96), (1, 257, 131, 96), (1, 14, 577, 96), (1, 24, 768, 96), (1, 257, 80, 128), (1, 160, 128, 128),
    (1, 160, 131, 128), (1, 257, 131, 128), (1, 5, 1031, 128), (1, 24, 912, 128),
]
WIDE = [(1, 1, 4, 4), (1, 1, 8, 16), (1, 1, 131, 16), (1, 640, 8, 40), (1, 60, 71, 40), (1, 257, 8, 72), (1, 1, 8, 72), (1, 8, 257, 72), (1, 160, 8, 130), (1, 33, 131, 130), (1, 490, 53, 64)]


@pytest.fixture(scope="module")
def M():
    import paper_2111_11124_amd as m
    assert torch.cuda.is_available(), "these tests need the MI355X"
    m.lib()
    return m


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16], ids=["f16", "bf16"])
@pytest.mark.parametrize("B,H,N,Dh", SIXTEEN)
def test_attention_products_by_every_kernel(M, B, H, N, Dh, dtype):
    run(M, B, H, N, Dh, dtype, False)


@pytest.mark.parametrize("large", [False, True], ids=["", "large"])
@pytest.mark.parametrize("B,H,N,Dh", WIDE)
def test_attention_products_by_every_kernel_binary32(M, B, H, N, Dh, large):
    run(M, B, H, N, Dh, torch.float32, large)


def test_attention_products_by_the_general_kernel_over_the_range_of_binary32(M):
    """Heads on scales of their own, too many of them for the kernel of few heads."""
    from tests.test_gpu_binary32_range import test_attention_products_over_the_range_of_binary32 as over_the_range
    over_the_range(M, 600, 64)
