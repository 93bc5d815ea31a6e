"""The backward walk at the edges of its rounds: lists around the checkpoint chunk (256) and
the shortest chunked list (512), of particles that touch every 4x4 sub-block of their tiles,
so that a round's pairs exceed its capacity and it keeps only its first entries (around 37
entries isotropic, 27 anisotropic); and scenes of which part lies behind opaque particles, so
that entries and whole chunks have no gradient record. Against the FP64 oracle, at the
tolerance of its other gradient comparisons: 1e-3 |g| + 1e-4 max|g| (FP32 sums of a few hundred
pixels and entries, transmittance recovered by division along at most one list)."""
import numpy as np
import pytest

import oracle as O
import scenegen as S

from tests import _helpers as TH

pytestmark = pytest.mark.gpu


def _stack(n, seed, opaque):
    """n wide particles one behind the other; with `opaque`, the front few stop every pixel."""
    rng = np.random.default_rng(seed)
    pos = np.stack([rng.uniform(-0.05, 0.05, n), rng.uniform(-0.05, 0.05, n), np.linspace(0.4, -0.4, n)])
    opacity = rng.uniform(0.010, 0.012, n)
    if opaque:
        opacity[:8] = 0.95
    return S.Scene(pos.astype(np.float32), np.full(n, 3.0, np.float32), opacity.astype(np.float32),
                   rng.uniform(0, 1, (3, n)).astype(np.float32), 0)


@pytest.mark.parametrize("family", ["iso", "aniso"])
@pytest.mark.parametrize("n,opaque", [(26, False), (28, False), (36, False), (38, False), (255, False), (257, False),
                                      (511, False), (513, False), (600, True), (1100, True)])
def test_rounds_match_oracle(family, n, opaque):
    import torch
    import paper_2403_14244_amd as P
    print(f"[gpu-case] bwd rounds {family} {n} {opaque}", flush=True)
    sc = _stack(n, n, opaque)
    an = family == "aniso"
    cam = S.look_at_camera((0.0, 0.0, 3.0), width=29, height=21)
    rng = np.random.default_rng(n)
    if an:
        sc = S.aniso_from_iso(sc)
        sc.rot[:] = rng.normal(size=sc.rot.shape)
        sc.scale *= rng.uniform(0.9, 1.1, sc.scale.shape).astype(np.float32)
    render = O.aniso64.render_aniso_views if an else O.render_views
    flags = render([sc], [cam], rounded=True)[3]
    W = (rng.normal(size=(3, cam.height, cam.width)) * ~flags[0][None]).astype(np.float32)
    assert flags[0].mean() < 0.2   # most pixels carry a weight
    R = (P.AnisoRasterizer if an else P.Rasterizer)()
    gs = (P.AnisoGaussianScene if an else P.GaussianScene).from_host(sc)
    _, st = R.render([gs], [cam], checkpoints=True)
    dL = torch.from_numpy(W.ravel().copy()).cuda()
    args = ([gs], [cam], st["fp"], st["bins"], (0.0, 0.0, 0.0), dL, st["T"], st["n_last"])
    ref = (O.aniso64.scene_grads_aniso if an else O.scene_grads)(sc, [cam], [W.astype(np.float64)])
    for what, kw in (("chunks", dict(image=st["image"], ckpt=st["ckpt"])), ("whole", {})):
        g = R.render_bwd(*args, **kw)[0]
        for name in ("pos", "scale", "opacity", "color") + (("rot",) if an else ()):
            TH.grad_check(getattr(g, name).cpu().numpy(), ref[name], f"{family} {n} {what} {name}")
