"""The loss kernels at the edges of their 32 x 22 output tiles, against the FP64 oracle.

Noise images in [0, 1]: local variances near 1/12, so the derivative maps' denominators are
far from C1 C2 and FP32 sums of 121 products stay within 1e-5 of the mean and 1e-4 of the
largest gradient (one gradient adds 121 map values, each within a few FP32 ulps)."""
import numpy as np
import pytest

from oracle import ssim64 as Q

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(1, 1, 1), (2, 22, 32), (1, 23, 33), (3, 21, 31), (1, 44, 64), (2, 45, 97),
                                   (1, 5, 130), (1, 130, 5)])
def test_loss_at_tile_edges(shape):
    import torch
    import paper_2403_14244_amd as P
    print(f"[gpu-case] loss tiles {shape}", flush=True)
    rng = np.random.default_rng(sum(shape))
    y = rng.uniform(0, 1, shape).astype(np.float32)
    x = np.clip(y + rng.normal(0, 0.2, shape), 0, 1).astype(np.float32)
    lref, gref = Q.l1_ssim_loss64(x, y)
    xt = torch.from_numpy(x).cuda().requires_grad_(True)
    yt = torch.from_numpy(y).cuda()
    loss = P.l1_ssim_loss(xt, yt)
    loss.backward()
    assert abs(float(loss.detach()) - lref) <= 1e-5
    assert np.abs(xt.grad.cpu().numpy() - gref).max() <= 1e-4 * np.abs(gref).max()
    assert abs(float(P.ssim(xt.detach(), yt)) - Q.ssim64(x, y)) <= 1e-5
