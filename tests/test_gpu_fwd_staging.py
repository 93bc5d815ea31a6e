"""The forward walk at the edges of its staging: batches of 1, 64, 65, 256, 257 and 513 entries
that reach every 4x4 sub-block of their tiles (full lists, waves without an entry, a last batch
of one), with and without pixels that stop before the next batch, on images that end inside a
tile and a sub-block and on one whose queue is longer than a dispatch group and not a multiple
of it. Against the FP64 oracle at the tolerance of its other image comparisons, its flagged
pixels held to one of their valid outcomes."""
import numpy as np
import pytest

import oracle as O
import scenegen as S

from tests import _helpers as TH

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("width,height", [(1, 1), (29, 21), (70, 18), (1037, 71)])
@pytest.mark.parametrize("n,opaque", [(1, False), (64, False), (65, False), (256, True), (257, True), (513, False)])
def test_batch_edges_match_oracle(n, opaque, width, height):
    import torch
    import paper_2403_14244_amd as P
    print(f"[gpu-case] fwd staging {n} {opaque} {width}x{height}", flush=True)
    rng = np.random.default_rng(n)
    pos = np.stack([rng.uniform(-0.05, 0.05, n), rng.uniform(-0.05, 0.05, n), np.linspace(0.4, -0.4, n)])
    opacity = rng.uniform(0.010, 0.012, n)
    if opaque:
        opacity[20:40] = 0.6
    sc = S.Scene(pos.astype(np.float32), np.full(n, 3.0, np.float32), opacity.astype(np.float32),
                 rng.uniform(0, 1, (3, n)).astype(np.float32), 0)
    cams = [S.look_at_camera((0.0, 0.0, 3.0), width=width, height=height)]
    bg = (0.2, 0.1, 0.3)
    R = P.Rasterizer()
    g = P.GaussianScene.from_host(sc)
    fp = R.project([g], cams)
    b = R.bin_sort(fp, [g.n], cams)
    ores = O.render_views([sc], cams, bg=bg, rounded=True)
    outs = TH.projected_outcomes(ores[4], cams, ores[5], bg)
    for what, (img, T, nl) in (("plain", R.render_fwd(fp, [g.n], b, cams, bg)),
                               ("ordered", R.render_fwd_ordered(fp, [g.n], b, cams, bg)),
                               ("wide", R.render_fwd_ordered(fp, [g.n], b, cams, bg, wide=True))):
        torch.cuda.synchronize()
        TH.check_image(img.cpu().numpy().reshape(3, height, width), T.cpu().numpy().reshape(height, width),
                       ores[0][0], ores[1][0], ores[3][0], outs[0], max_flag_frac=0.06,
                       what=f"{n} {width}x{height} {what}")
        keep = ~ores[3][0]
        np.testing.assert_array_equal(nl.cpu().numpy().reshape(height, width)[keep], ores[2][0][keep])
