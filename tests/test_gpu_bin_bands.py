"""Binning of views larger than the tiles a workgroup counts at once, bit for bit against the
oracle's binning."""
import numpy as np
import pytest

import oracle as O
import scenegen as S
from tests import _helpers as TH

pytestmark = pytest.mark.gpu


def _footprints(n, w, h, seed, r_max, big=0.02):
    """Disks of up to r_max pixels, a share `big` of them of up to eight times as many."""
    rng = np.random.default_rng(seed)
    u, v = rng.uniform(-0.1 * w, 1.1 * w, n), rng.uniform(-0.1 * h, 1.1 * h, n)
    r = np.where(rng.uniform(size=n) < big, rng.uniform(0, 8 * r_max, n), rng.uniform(0, r_max, n))
    f = lambda a: a.astype(np.float32)
    return TH.synthetic_f32_footprints(f(u), f(v), f(rng.uniform(0.5, 9.0, n)), f(r), w, h, seed=seed)


def _cams(sizes):
    return [S.look_at_camera((0, 0, 3), width=w, height=h) for w, h in sizes]


def _check(bins, ob):
    import torch
    torch.cuda.synchronize()
    n = bins.n_entries()
    assert n == ob.keys.shape[0]
    np.testing.assert_array_equal(bins.pidx[:n].cpu().numpy().view(np.uint32), ob.pidx)
    np.testing.assert_array_equal(bins.ranges.cpu().numpy().view(np.uint32), ob.ranges)
    np.testing.assert_array_equal(bins.offsets.cpu().numpy().view(np.uint32), ob.offsets)


def test_static_scratch_too_small_for_the_matrix():
    """A capacity at which the static scratch holds neither the packed boxes nor all chunks' rows of
    the view's million tiles: fewer chunks."""
    import paper_2403_14244_amd as P
    n, w, h = 20_000, 16384, 16384
    views, cams = [_footprints(n, w, h, 91, 30.0)], _cams([(w, h)])
    ob = O.bin_sort_ref(views)
    print(f"[gpu-case] static scratch, 16384 x 16384: {ob.keys.shape[0]} entries", flush=True)
    bins = P.Rasterizer().bin_sort_static(TH.upload_footprints(views, ob), [n], cams, capacity=5_200_000)
    bins.verify()
    _check(bins, ob)
