"""Parameter gradients at every colour degree over one view (the anisotropic family's single-view
kernel), two, and 17 (a second launch of one view that adds to the first's sums), for particle
counts below, at and above a workgroup. Against the FP64 oracle, at the tolerance of its other
gradient comparisons: 1e-3 |g| + 1e-4 max|g|."""
import math

import numpy as np
import pytest

import oracle as O
import scenegen as S

from tests import _helpers as TH

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("family", ["iso", "aniso"])
@pytest.mark.parametrize("deg,views,n", [(0, 1, 256), (1, 1, 100), (2, 1, 257), (3, 1, 300), (2, 2, 257), (3, 2, 300),
                                         (3, 17, 60), (0, 17, 60)])
def test_gradients_match_oracle(family, deg, views, n):
    import torch
    import paper_2403_14244_amd as P
    print(f"[gpu-case] grad views {family} {deg} {views} {n}", flush=True)
    rng = np.random.default_rng(1000 + 100 * deg + views)
    base = S.uniform_cube_scene(n, seed=deg + views, log_scale_mean=math.log(0.05), log_scale_std=0.4)
    color = rng.normal(0, 0.1, (3 * (deg + 1) ** 2, n)).astype(np.float32)
    color[:3] = base.color[:3]
    sc = S.Scene(base.pos, base.scale, base.opacity, color, deg)
    cams = [S.look_at_camera((0.6 * math.sin(0.37 * i), 0.2, 3.0 + 0.05 * i), width=40, height=33) for i in range(views)]
    an = family == "aniso"
    if an:
        sc = S.aniso_from_iso(sc)
        sc.rot[:] = rng.normal(size=sc.rot.shape)
        sc.scale *= rng.uniform(0.6, 1.6, sc.scale.shape).astype(np.float32)
    render = O.aniso64.render_aniso_views if an else O.render_views
    flags = render([sc] * views, cams, rounded=True)[3]
    Ws = [(rng.normal(size=(3, c.height, c.width)) * ~f[None]).astype(np.float32) for c, f in zip(cams, flags)]
    assert np.mean([f.mean() for f in flags]) < 0.05   # nearly all pixels carry a weight
    R = (P.AnisoRasterizer if an else P.Rasterizer)()
    gs = (P.AnisoGaussianScene if an else P.GaussianScene).from_host(sc)
    _, st = R.render([gs] * views, cams)
    dL = torch.from_numpy(np.concatenate([w.ravel() for w in Ws])).cuda()
    g = R.render_bwd([gs] * views, cams, st["fp"], st["bins"], (0.0, 0.0, 0.0), dL, st["T"], st["n_last"])[0]
    ref = (O.aniso64.scene_grads_aniso if an else O.scene_grads)(sc, cams, [w.astype(np.float64) for w in Ws])
    for name in ("pos", "scale", "opacity", "color") + (("rot",) if an else ()):
        TH.grad_check(getattr(g, name).cpu().numpy(), ref[name], f"{family} {deg} {views} {name}")
