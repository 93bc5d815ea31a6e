"""Gradients of kernels narrower than a pixel, and of thin ones at an angle to the pixel grid,
particle by particle, against the FP64 oracle. A particle's sum over pixels of (weight) x
(offset from its centre)^2 is then far smaller than the offsets from any other origin squared, so
that sums formed about the tile or the sub-block and moved to the centre lose it.

Narrow kernels: one particle per 3 x 3 pixels, dL/dimage positive and the background black, so that
the terms of a scale, opacity or colour gradient do not cancel and each is compared by itself. The
bound is what the centre's FP32 rounding allows: with each coordinate off by up to half an ulp h, d^2
at a distance d from a pixel is off by 2 sqrt(2) h / d of itself (d: the nearest pixel), and
exp(-d^2 / s^2) by at most 2 sqrt(2) h 2.35 / s (alpha reaches 1/255 at d = 2.35 s); twice that, and
2e-5 for the sums and powers of FP32. Both families (anisotropic: three equal axes, and the gradient
along all three together, the sum of s_k dL/ds_k). Thin kernels (4.5 x 0.15 pixels and
the like): the exponent sums terms of up to (7 / 0.15)^2 / 2 with 2^-24 of each, 1.3e-4, and the narrow
axis' gradient is what is left of second moments (4.5 / 0.15)^2 = 900 times as large with 2^-24 of
each and a few roundings, 2e-4: 2e-3 as the root mean square over the particles, few of which overlap."""
import numpy as np
import pytest

import oracle as O
import scenegen as S

pytestmark = pytest.mark.gpu


def _place(rng, cam, pitch, offset):
    """World centres whose images lie `offset` [2, n] from the middle of a pixel, one per pitch^2."""
    k = np.arange(pitch // 2, cam.width - pitch // 2, pitch)
    i, j = (a.ravel() for a in np.meshgrid(k, k))
    off = offset(i.size)
    z = rng.permutation(np.linspace(2.6, 3.4, i.size))
    p = np.stack([(i + 0.5 + off[0] - cam.cx) * z / cam.f, (j + 0.5 + off[1] - cam.cy) * z / cam.f, z])
    return (cam.R.astype(np.float64).T @ (p - cam.t.astype(np.float64)[:, None])).astype(np.float32), z


def _weights(rng, flags, cam):
    return (rng.uniform(0.5, 1.5, (3, cam.height, cam.width)) * ~flags[None]).astype(np.float32)


def _gpu(sc, cam, W, an):
    import torch
    import paper_2403_14244_amd as P
    R = (P.AnisoRasterizer if an else P.Rasterizer)()
    gs = (P.AnisoGaussianScene if an else P.GaussianScene).from_host(sc)
    _, st = R.render([gs], [cam], checkpoints=True)
    g = R.render_bwd([gs], [cam], st["fp"], st["bins"], (0.0, 0.0, 0.0), torch.from_numpy(W.ravel().copy()).cuda(),
                     st["T"], st["n_last"], image=st["image"], ckpt=st["ckpt"])[0]
    return {k: getattr(g, k).cpu().numpy().astype(np.float64)
            for k in ("pos", "scale", "opacity", "color") + (("rot",) if an else ())}


def _rms(a):
    return float(np.sqrt((a * a).mean()))


@pytest.mark.parametrize("family", ["iso", "aniso"])
@pytest.mark.parametrize("s_px", [0.05, 0.1, 0.2, 0.4])
def test_kernels_narrower_than_a_pixel(family, s_px):
    rng = np.random.default_rng(int(100 * s_px))
    cam = S.look_at_camera((0.0, 0.0, 3.0), width=32, height=32)

    def offset(n):
        r, a = np.exp(rng.uniform(np.log(0.004), np.log(1.8 * s_px), n)), rng.uniform(0, 2 * np.pi, n)
        return np.stack([r * np.cos(a), r * np.sin(a)])
    pos, z = _place(rng, cam, 3, offset)
    n = pos.shape[1]
    sc = S.Scene(pos, (s_px * z / cam.f).astype(np.float32), rng.uniform(0.3, 0.9, n).astype(np.float32),
                 rng.uniform(0.2, 1, (3, n)).astype(np.float32), 0)
    an = family == "aniso"
    if an:
        sc = S.aniso_from_iso(sc)
        sc.rot[:] = rng.normal(size=sc.rot.shape)
    print(f"[gpu-case] small kernels {family} {s_px}: {n}", flush=True)
    res = (O.aniso64.render_aniso_views if an else O.render_views)([sc], [cam], rounded=True)
    W, pr = _weights(rng, res[3][0], cam), res[4][0]
    ref = (O.aniso64.scene_grads_aniso if an else O.scene_grads)(sc, [cam], [W.astype(np.float64)])
    got = _gpu(sc, cam, W, an)
    if an:
        for g in (ref, got):
            g["scale"] = (g["scale"] * sc.scale.astype(np.float64)).sum(0)
    h = np.spacing(np.float32(max(cam.width, cam.height) - 1)) / 2
    d = np.hypot(pr.u - np.floor(pr.u) - 0.5, pr.v - np.floor(pr.v) - 0.5)
    bound = 2 * 2 * np.sqrt(2) * h * (1 / d + 2.35 / s_px) + 2e-5
    assert (np.abs(ref["scale"]) > 0).all() and bound.max() < 2.5e-3
    for name in ("scale", "opacity", "color"):
        err = np.abs(got[name] - ref[name]) / np.abs(ref[name])
        assert (err <= bound).all(), (name, float(err.max()), float((err / bound).max()))
    assert _rms(got["pos"] - ref["pos"]) <= 1e-3 * _rms(ref["pos"])


@pytest.mark.parametrize("narrow,ratio,degrees", [(0.15, 30.0, 45.0), (0.3, 20.0, 45.0), (0.3, 20.0, 20.0)])
def test_thin_kernels_at_an_angle(narrow, ratio, degrees):
    rng = np.random.default_rng(int(1000 * narrow + degrees))
    cam = S.look_at_camera((0.0, 0.0, 3.0), width=60, height=60)
    pos, z = _place(rng, cam, 12, lambda n: rng.uniform(-0.3, 0.3, (2, n)))
    n = pos.shape[1]
    turn = np.radians(degrees + rng.uniform(-3, 3, n))
    zero = np.zeros(n)
    sc = S.AnisoScene(pos=pos, rot=np.stack([np.cos(turn / 2), zero, zero, np.sin(turn / 2)]).astype(np.float32),
                      scale=np.stack([narrow * ratio * z / cam.f, narrow * z / cam.f, narrow * z / cam.f]).astype(np.float32),
                      opacity=rng.uniform(0.3, 0.9, n).astype(np.float32),
                      color=rng.uniform(0.2, 1, (3, n)).astype(np.float32), sh_degree=0)
    print(f"[gpu-case] thin kernels {narrow} x {narrow * ratio} at {degrees}: {n}", flush=True)
    flags = O.aniso64.render_aniso_views([sc], [cam], rounded=True)[3][0]
    W = _weights(rng, flags, cam)
    ref = O.aniso64.scene_grads_aniso(sc, [cam], [W.astype(np.float64)])
    got = _gpu(sc, cam, W, True)
    # (the third axis points at the eye: next to no gradient)
    for name, a, b in (("long axis", got["scale"][0], ref["scale"][0]), ("narrow axis", got["scale"][1], ref["scale"][1])) + tuple(
            (k, got[k], ref[k]) for k in ("rot", "pos", "opacity", "color")):
        assert _rms(a - b) <= 2e-3 * _rms(b), (name, _rms(a - b) / _rms(b))
