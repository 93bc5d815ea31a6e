"""Workspace sizes of the loss calls up to the largest accepted images: three derivative maps, and a
block sum per 32 x 22 tile (two for the loss), however long a row or a column is."""
import ctypes

import pytest


@pytest.mark.parametrize("channels,height,width", [(3, 1080, 1920), (1, 1, 2 ** 31 - 1), (1, 1, 2 ** 31 - 20),
                                                   (1, 2 ** 31 - 1, 1), (1, 2 ** 31 - 22, 1), (65535, 1, 32767)])
def test_workspace_sizes(channels, height, width):
    from paper_2403_14244_amd import _abi as A
    up = lambda x: (x + 255) // 256 * 256
    n, blocks = channels * height * width, channels * -(-width // 32) * -(-height // 22)
    need = ctypes.c_size_t(0)
    A.check(A.lib().isogs_ssim_fwd(None, None, channels, height, width, None, None, ctypes.byref(need), None))
    assert need.value == 3 * up(4 * n) + up(8 * blocks)
    A.check(A.lib().isogs_loss_fwd(None, None, channels, height, width, 0.2, None, None, ctypes.byref(need), None))
    assert need.value == 3 * up(4 * n) + 2 * up(8 * blocks)
