"""Launches whose workgroups loop: more long tiles than the wide forward starts workgroups for,
and more chunks of them than the backward does. Every tile of a 66 x 65 tile image holds all 2100
particles. The backward at a capacity for which it loops equals the one at a capacity for which
it does not, bit for bit; the forward equals the one-wave-per-quadrant walk up to rounding: 2e-5
as in the other comparisons of the two walks, and 1.2e-4 where T passes within rounding of the
threshold (the light that 1e-4 of transmittance lets through)."""
import numpy as np
import pytest

import scenegen as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("family", ["iso", "aniso"])
def test_looping_launches(family):
    import torch
    import paper_2403_14244_amd as P
    print(f"[gpu-case] large launch {family}", flush=True)
    n, width, height = 2100, 1051, 1037
    rng = np.random.default_rng(5)
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
    for capacity in (9_500_000, 18_000_000):
        fp = R.project([g], cams)
        b = R.bin_sort(fp, [g.n], cams, capacity=capacity)
        lens = b.ranges[:, 1] - b.ranges[:, 0]
        assert b.capacity == capacity and int(lens.min()) >= 2048
        ck = R.checkpoint_buffer(b)
        img, T, nl = R.render_fwd_ordered(fp, [g.n], b, cams, (0.1, 0.2, 0.3), ckpt=ck, wide=True)
        gr = R.render_bwd([g], cams, fp, b, (0.1, 0.2, 0.3), dL, T, nl, image=img, ckpt=ck)[0]
        seq = R.render_fwd_ordered(fp, [g.n], b, cams, (0.1, 0.2, 0.3))
        torch.cuda.synchronize()
        res.append([img, T, nl] + [getattr(gr, k) for k in ("pos", "scale", "opacity", "color")])
        d = (img - seq[0]).abs().reshape(3, -1).amax(0)
        assert float(d.max()) <= 1.2e-4 and float((d > 2e-5).float().mean()) < 0.01
        assert float((nl == seq[2]).float().mean()) > 0.99
        assert int(((nl.reshape(-1).max()) + 255) // 256) * lens.numel() > 32768   # a second turn for some
    for x, y in zip(*res):
        assert torch.equal(x, y)
