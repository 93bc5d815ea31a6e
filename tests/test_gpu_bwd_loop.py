"""The backward of launches whose workgroups loop (more than 327680 possible items), bit for bit the
one of a capacity for which they do not: a tile's gradients do not depend on which workgroup takes
it. Every tile of a 66 x 65 tile image holds all 2100 particles, so that there are more items
(4290 tiles of up to nine chunks) than workgroups, and some take a second one."""
import numpy as np
import pytest

import scenegen as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("family", ["iso", "aniso"])
def test_looping_backward(family):
    import torch
    import paper_2403_14244_amd as P
    print(f"[gpu-case] bwd loop {family}", flush=True)
    n, width, height = 2100, 1051, 1037
    rng = np.random.default_rng(6)
    pos = np.stack([rng.uniform(-0.05, 0.05, n), rng.uniform(-0.05, 0.05, n), np.linspace(0.4, -0.4, n)])
    sc = S.Scene(pos.astype(np.float32), np.full(n, 30.0, np.float32),
                 rng.uniform(0.0042, 0.006, n).astype(np.float32), rng.uniform(0, 1, (3, n)).astype(np.float32), 0)
    an = family == "aniso"
    if an:
        sc = S.aniso_from_iso(sc)
    cams = [S.look_at_camera((0.0, 0.0, 3.0), width=width, height=height)]
    R = (P.AnisoRasterizer if an else P.Rasterizer)()
    g = (P.AnisoGaussianScene if an else P.GaussianScene).from_host(sc)
    dL = torch.from_numpy(rng.normal(size=3 * height * width).astype(np.float32)).cuda()
    res = []
    for capacity in (9_500_000, 84_000_000):
        fp = R.project([g], cams)
        b = R.bin_sort(fp, [g.n], cams, capacity=capacity)
        tiles = b.ranges.shape[0]
        assert b.capacity == capacity and (tiles + capacity // 256 + 1 > 327680) == (len(res) == 1)
        ck = R.checkpoint_buffer(b)
        img, T, nl = R.render_fwd_ordered(fp, [g.n], b, cams, ckpt=ck)
        assert tiles * ((int(nl.max()) + 255) // 256) > 32768
        gr = R.render_bwd([g], cams, fp, b, (0.0, 0.0, 0.0), dL, T, nl, image=img, ckpt=ck)[0]
        torch.cuda.synchronize()
        res.append([getattr(gr, k) for k in ("pos", "scale", "opacity", "color") + (("rot",) if an else ())])
    for x, y in zip(*res):
        assert torch.equal(x, y)
