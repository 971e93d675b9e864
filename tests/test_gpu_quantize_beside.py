"""quantize_qkv where heads of up to 1 MB next to the rows of Q and K change from parts to whole (64 heads of 2-byte elements, 80 of
4-byte ones), both sides of the line: the codes and scales of the other calls, bit for bit."""
import pytest

torch = pytest.importorskip("torch")

import test_gpu_quantize_heads as heads_test

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16, torch.float32])
@pytest.mark.parametrize("heads,N,d", [(63, 1777, 128), (64, 1777, 128), (64, 4096, 128), (64, 4097, 128), (79, 4096, 64), (80, 4096, 64), (80, 4097, 64)])
def test_both_sides_of_the_line(heads, N, d, dtype):
    heads_test.test_headwise_codes_and_scales(heads, N, d, dtype)
