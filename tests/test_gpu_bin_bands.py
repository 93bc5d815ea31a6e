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


# eight lanes per particle: few particles, or a capacity of 16 entries per particle
CASES = {
    "nine_bands": lambda: ([(_footprints(6000, 12288, 6912, 1, 60.0), 12288, 6912), (_footprints(300, 40, 30, 2, 8.0), 40, 30),
                            (_footprints(900, 7000, 1600, 3, 40.0), 7000, 1600)], 0),
    "many_bands": lambda: ([(_footprints(3000, 32768, 8192, 4, 300.0), 32768, 8192)], 0),
    "many_particles": lambda: ([(_footprints(140_000, 7680, 4320, 5, 12.0, 0.01), 7680, 4320)], 0),
    "many_particles_nine_bands": lambda: ([(_footprints(140_000, 12288, 6912, 6, 20.0, 0.01), 12288, 6912)], 0),
    "large_capacity": lambda: ([(_footprints(140_000, 12288, 6912, 7, 20.0, 0.01), 12288, 6912)], 16),
    "two_views": lambda: ([(_footprints(100_000, 5120, 2880, 8, 12.0, 0.01), 5120, 2880),
                           (_footprints(60_000, 4096, 4096, 9, 12.0, 0.01), 4096, 4096)], 0),
}


@pytest.mark.parametrize("case", list(CASES))
def test_bands_are_bit_exact(case):
    import paper_2403_14244_amd as P
    made, per = CASES[case]()
    views, cams = [m[0] for m in made], _cams([m[1:] for m in made])
    npv = [v["u"].shape[0] for v in views]
    ob = O.bin_sort_ref(views)
    capacity = max(ob.keys.shape[0] + 5, per * sum(npv))
    print(f"[gpu-case] bands {case}: {ob.keys.shape[0]} entries", flush=True)
    _check(P.Rasterizer().bin_sort(TH.upload_footprints(views, ob), npv, cams, capacity=capacity), ob)


@pytest.mark.parametrize("n", [1200, 140_000])
def test_tile_counts_that_disagree_in_bands(n):
    """A particle has the first `tile_count` of its member tiles (row-major), whichever bands they
    lie in; entries beyond its members belong to no tile and follow all others, by particle."""
    import torch
    import paper_2403_14244_amd as P
    w, h = 7680, 4320
    views, cams = [_footprints(n, w, h, 92, 150.0 if n < 2000 else 12.0, 0.05 if n < 2000 else 0.01)], _cams([(w, h)])
    ob = O.bin_sort_ref(views)
    rng = np.random.default_rng(93)
    have = ob.tile_count.astype(np.int64)
    off = rng.integers(-2, 3, n) * np.where(rng.uniform(size=n) < 0.5, 1, 1 + have // 3)
    want = np.where(rng.uniform(size=n) < 0.3, np.maximum(0, have + off), have)
    order = np.lexsort((ob.keys >> np.uint64(32), ob.pidx))   # the members in emit order
    tile, who = (ob.keys >> np.uint64(32)).astype(np.int64)[order], ob.pidx.astype(np.int64)[order]
    first = np.concatenate([[0], np.cumsum(have)])[:-1]
    keep = np.arange(who.size) - first[who] < want[who]
    tile, who = tile[keep], who[keep]
    z = views[0]["z"].view(np.uint32).astype(np.int64)
    expect = np.concatenate([who[np.lexsort((who, z[who], tile))], np.repeat(np.arange(n), np.maximum(0, want - have))])
    fp = TH.upload_footprints(views, ob)
    fp.tile_count.copy_(torch.from_numpy(want.astype(np.int32)))
    print(f"[gpu-case] tile counts in bands {n}: {expect.size} entries", flush=True)
    spans = (ob.ranges[:, 1] > 0).reshape(-1, (w + 15) // 16).any(1).sum()
    assert spans > 3 * 76 and (want > have).sum() > 50 and (want < have).sum() > 50   # rows of every band
    bins = P.Rasterizer().bin_sort(fp, [n], cams)
    assert bins.n_entries() == expect.size
    np.testing.assert_array_equal(bins.pidx[:expect.size].cpu().numpy().astype(np.int64), expect)
    np.testing.assert_array_equal(bins.offsets.cpu().numpy().astype(np.int64), np.concatenate([[0], np.cumsum(want)])[:-1])
    len_ = np.bincount(tile, minlength=ob.ranges.shape[0])
    end = np.cumsum(len_)
    np.testing.assert_array_equal(bins.ranges.cpu().numpy().astype(np.int64),
                                  np.where(len_[:, None] > 0, np.stack([end - len_, end], 1), 0))


def test_bands_without_the_packed_boxes():
    """17M particles, nearly all culled: the static scratch is too small for their boxes."""
    import torch
    import paper_2403_14244_amd as P
    n, w, h = 17_000_000, 5120, 2880
    views, cams = [_footprints(40_000, w, h, 94, 20.0)], _cams([(w, h)])
    ob = O.bin_sort_ref(views)
    small = TH.upload_footprints(views, ob)
    at = torch.randperm(n, generator=torch.Generator().manual_seed(1))[:40_000].sort().values.cuda()
    fp = P.Footprints(torch.zeros(n, 8, device="cuda"), torch.ones(n, device="cuda"),
                      torch.zeros(n, dtype=torch.int32, device="cuda"))
    fp.record[at], fp.depth[at], fp.tile_count[at] = small.record, small.depth, small.tile_count
    print("[gpu-case] bands, static scratch, 17M particles", flush=True)
    bins = P.Rasterizer().bin_sort_static(fp, [n], cams, capacity=ob.keys.shape[0] + 7)
    bins.verify()
    e = bins.n_entries()
    assert e == ob.keys.shape[0]
    np.testing.assert_array_equal(bins.pidx[:e].cpu().numpy().astype(np.int64),
                                  at.cpu().numpy()[ob.pidx.astype(np.int64)])
    np.testing.assert_array_equal(bins.ranges.cpu().numpy().view(np.uint32), ob.ranges)
