"""Binning paths chosen by size, bit for bit against the oracle's binning: views of more tiles
than a workgroup counts at once (the larger band, and several bands), calls of more particles
than share lanes, boxes on both sides of the packed 4 x 4 form, equal depths in every size class
of the segment sort, tile counts that disagree with the footprints, and the static scratch where
it is too small for the packed boxes."""
import numpy as np
import pytest

import oracle as O
import scenegen as S
from tests import _helpers as TH

pytestmark = pytest.mark.gpu


def _footprints(n, w, h, seed, r_max, depths=None, big=0.02):
    rng = np.random.default_rng(seed)
    u, v = rng.uniform(-20, w + 20, n), rng.uniform(-20, h + 20, n)
    r = np.where(rng.uniform(size=n) < big, rng.uniform(0, 4 * r_max, n), rng.uniform(0, r_max, n))
    z = rng.uniform(0.5, 9.0, n) if depths is None else rng.choice(np.asarray(depths), n)
    f = lambda a: a.astype(np.float32)
    return TH.synthetic_f32_footprints(f(u), f(v), f(z), f(r), w, h, seed=seed)


def _crowd(n, seed, depths):
    u, v, z, r = S.crowded_projected(n, 48, 32, 24.0, 8.0, 2.0, seed=seed, max_radius=0.5, depths=depths)
    return TH.synthetic_f32_footprints(u, v, z, r, 48, 32, seed=seed)


CASES = {
    "large_band": lambda: [(_footprints(5000, 2600, 1700, 1, 30.0), 2600, 1700), (_footprints(300, 40, 30, 2, 8.0), 40, 30)],
    "four_bands": lambda: [(_footprints(4000, 7680, 4320, 3, 60.0), 7680, 4320)],
    "large_band_ungrouped": lambda: [(_footprints(140_000, 2600, 1700, 4, 20.0), 2600, 1700)],
    "ungrouped": lambda: [(_footprints(70_000, 500, 400, 5, 9.0), 500, 400), (_footprints(70_000, 333, 217, 6, 9.0), 333, 217)],
    "seventeen_views": lambda: [(_footprints(700 + 13 * k, 90 + k, 70 + 3 * k, 7 + k, 10.0), 90 + k, 70 + 3 * k)
                                for k in range(17)],
    "equal_depths": lambda: [(_crowd(n, 30 + k, [2.5]), 48, 32) for k, n in enumerate((65, 256, 257, 1024, 1025, 4096, 4097, 9000))],
    "two_depths": lambda: [(_crowd(n, 50 + k, [2.5, 2.75]), 48, 32) for k, n in enumerate((200, 900, 3000, 12000))],
}


def _cams(sizes):
    return [S.look_at_camera((0, 0, 3), width=w, height=h) for w, h in sizes]


@pytest.mark.parametrize("case", list(CASES))
def test_binning_is_bit_exact(case):
    import torch
    import paper_2403_14244_amd as P
    made = CASES[case]()
    views, cams = [m[0] for m in made], _cams([m[1:] for m in made])
    ob = O.bin_sort_ref(views)
    print(f"[gpu-case] binning {case}: {ob.keys.shape[0]} entries", flush=True)
    R = P.Rasterizer()
    bins = R.bin_sort(TH.upload_footprints(views, ob), [v["u"].shape[0] for v in views], cams, with_keys=True)
    torch.cuda.synchronize()
    n = bins.n_entries()
    assert n == ob.keys.shape[0]
    np.testing.assert_array_equal(bins.keys[:n].cpu().numpy().view(np.uint64), ob.keys)
    np.testing.assert_array_equal(bins.pidx[:n].cpu().numpy().view(np.uint32), ob.pidx)
    np.testing.assert_array_equal(bins.ranges.cpu().numpy().view(np.uint32), ob.ranges)
    np.testing.assert_array_equal(bins.offsets.cpu().numpy().view(np.uint32), ob.offsets)


@pytest.mark.parametrize("n", [900, 140_000])
def test_tile_counts_that_disagree(n):
    """A particle has the first `tile_count` of its member tiles (row-major); entries beyond its
    members belong to no tile and follow all others, by particle."""
    import torch
    import paper_2403_14244_amd as P
    w, h = 300, 200
    views, cams = [_footprints(n, w, h, 77, 12.0)], _cams([(w, h)])
    ob = O.bin_sort_ref(views)
    rng = np.random.default_rng(78)
    have = ob.tile_count.astype(np.int64)
    want = np.where(rng.uniform(size=n) < 0.3, np.maximum(0, have + rng.integers(-2, 3, n)), have)
    # the members of each particle in emit order, from the oracle's sorted keys
    order = np.lexsort((ob.keys >> np.uint64(32), ob.pidx))
    tile, who = (ob.keys >> np.uint64(32)).astype(np.int64)[order], ob.pidx.astype(np.int64)[order]
    first = np.concatenate([[0], np.cumsum(have)])[:-1]
    keep = np.arange(who.size) - first[who] < want[who]
    tile, who = tile[keep], who[keep]
    z = views[0]["z"].view(np.uint32).astype(np.int64)
    by = np.lexsort((who, z[who], tile))
    missing = np.repeat(np.arange(n), np.maximum(0, want - have))
    expect = np.concatenate([who[by], missing])
    fp = TH.upload_footprints(views, ob)
    fp.tile_count.copy_(torch.from_numpy(want.astype(np.int32)))
    print(f"[gpu-case] tile counts {n}: {expect.size} entries, {missing.size} without a tile", flush=True)
    assert missing.size > 50 and (want < have).sum() > 50
    bins = P.Rasterizer().bin_sort(fp, [n], cams)
    assert bins.n_entries() == expect.size
    np.testing.assert_array_equal(bins.pidx[:expect.size].cpu().numpy().astype(np.int64), expect)
    np.testing.assert_array_equal(bins.offsets.cpu().numpy().astype(np.int64), np.concatenate([[0], np.cumsum(want)])[:-1])
    T = ((w + 15) // 16) * ((h + 15) // 16)
    len_ = np.bincount(tile, minlength=T)
    end = np.cumsum(len_)
    np.testing.assert_array_equal(bins.ranges.cpu().numpy().astype(np.int64),
                                  np.where(len_[:, None] > 0, np.stack([end - len_, end], 1), 0))


def test_static_scratch_too_small_for_the_boxes():
    """17M particles, nearly all culled: the packed boxes alone (8 bytes each) exceed the static
    array; the call is made without them."""
    import torch
    import paper_2403_14244_amd as P
    n, w, h = 17_000_000, 640, 360
    views, cams = [_footprints(40_000, w, h, 90, 12.0)], _cams([(w, h)])
    ob = O.bin_sort_ref(views)
    small = TH.upload_footprints(views, ob)
    at = torch.randperm(n, generator=torch.Generator().manual_seed(1))[:40_000].sort().values.cuda()
    fp = P.Footprints(torch.zeros(n, 8, device="cuda"), torch.ones(n, device="cuda"),
                      torch.zeros(n, dtype=torch.int32, device="cuda"))
    fp.record[at], fp.depth[at], fp.tile_count[at] = small.record, small.depth, small.tile_count
    print("[gpu-case] static scratch, 17M particles", flush=True)
    bins = P.Rasterizer().bin_sort_static(fp, [n], cams, capacity=ob.keys.shape[0] + 7)
    bins.verify()
    e = bins.n_entries()
    assert e == ob.keys.shape[0]
    np.testing.assert_array_equal(bins.pidx[:e].cpu().numpy().astype(np.int64),
                                  at.cpu().numpy()[ob.pidx.astype(np.int64)])
    np.testing.assert_array_equal(bins.ranges.cpu().numpy().view(np.uint32), ob.ranges)
