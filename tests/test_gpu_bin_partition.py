"""Long tile segments, bit for bit against the oracle's binning: at the edges of the distribution's
LDS windows (14720 entries, up to four of them, one more), with a single depth held by more
entries than a window (written directly between windows), and with all depths equal."""
import numpy as np
import pytest

import oracle as O
import scenegen as S
from tests import _helpers as TH

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [4097, 14720, 14721, 29441, 58880, 58881, 70_000])
@pytest.mark.parametrize("depths", ["spread", "clump", "equal"])
def test_long_segments_are_bit_exact(n, depths):
    import torch
    import paper_2403_14244_amd as P
    print(f"[gpu-case] bin partition {n} {depths}", flush=True)
    rng = np.random.default_rng(n)
    z = rng.uniform(0.5, 9.0, n)
    if depths == "clump":
        z[rng.permutation(n)[: n // 2]] = 3.25
    if depths == "equal":
        z[:] = 2.5
    f = lambda a: a.astype(np.float32)
    # every particle reaches the one tile of its corner; few reach the neighbouring tile
    u, v, r = rng.uniform(2, 13, n), rng.uniform(2, 13, n), rng.uniform(1.0, 2.6, n)
    view = TH.synthetic_f32_footprints(f(u), f(v), f(z), f(r), 32, 16, seed=n)
    cams = [S.look_at_camera((0, 0, 3), width=32, height=16)]
    ob = O.bin_sort_ref([view])
    R = P.Rasterizer()
    bins = R.bin_sort(TH.upload_footprints([view], ob), [n], cams, with_keys=True)
    torch.cuda.synchronize()
    m = bins.n_entries()
    assert m == ob.keys.shape[0]
    np.testing.assert_array_equal(bins.keys[:m].cpu().numpy().view(np.uint64), ob.keys)
    np.testing.assert_array_equal(bins.pidx[:m].cpu().numpy().view(np.uint32), ob.pidx)
