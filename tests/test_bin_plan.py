"""The bin sort's plan, on the host: how many workgroups count and place a view, and how much
memory the call asks for, over image sizes on both sides of the tiles that a workgroup counts at
once (36864, a band) and over the capacities that the static scratch allows."""
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2403_14244_amd")
STATIC = 128 << 20
BAND = 36864

SOURCE = r"""
#include <cstdio>
#include <vector>
#include "kernels.h"
int main() {
    long long nv, n, w, h, cap, limit;
    while (scanf("%lld %lld %lld %lld %lld %lld", &nv, &n, &w, &h, &cap, &limit) == 6) {
        std::vector<int32_t> npv(nv, (int32_t)n);
        isogs_camera c{};
        c.width = (int32_t)w;
        c.height = (int32_t)h;
        std::vector<isogs_camera> cams(nv, c);
        const isogs::BinSortPlan p =
            isogs::plan_bin_sort(npv.data(), cams.data(), (int32_t)nv, (uint64_t)cap, limit ? (size_t)limit : SIZE_MAX);
        printf("%zu %u %d\n", p.bytes, p.chunks, (int)p.boxes);
    }
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    """plan([(views, particles per view, width, height, capacity, limit), ...]) -> [bytes, chunks, boxes]"""
    lib = os.path.join(PKG, "libisogs.so")
    if not os.path.exists(lib):
        pytest.skip("libisogs.so not built (run python paper_2403_14244_amd/build.py)")
    d = tmp_path_factory.mktemp("plan")
    src, exe = d / "plan.cpp", d / "plan"
    src.write_text(SOURCE)
    rocm = "/opt/rocm"
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", f"-I{rocm}/include", f"-I{PKG}/csrc", str(src), "-o",
                    str(exe), lib, f"-L{rocm}/lib", "-lamdhip64", f"-Wl,-rpath,{PKG}:{rocm}/lib"], check=True)

    def run(calls):
        text = "\n".join(" ".join(str(int(x)) for x in c) for c in calls)
        out = subprocess.run([str(exe)], input=text, capture_output=True, text=True, check=True).stdout
        return np.array([[int(x) for x in line.split()] for line in out.splitlines()])
    return run


def _tiles(w, h):
    return ((w + 15) // 16) * ((h + 15) // 16)


def _told(nv, n, w, h, cap):
    """The bytes that isogs.h states: 20 per entry and per tile and the sort's tables."""
    a = lambda x: (x + 255) // 256 * 256
    tiles, sort_tiles = nv * _tiles(w, h), (cap + 4095) // 4096
    long_max = min(tiles, cap // 16385 + 1)
    return (5 * a(4 * cap) + 2048 * sort_tiles + 1028 * (sort_tiles + long_max) + 40 * long_max + 20 * tiles +
            (nv * n + 2047) // 2048 * 4 + 40960)


def _groups(nv, n, w, h, chunks):
    return chunks * -(-_tiles(w, h) // BAND)


@pytest.mark.parametrize("n,w,h,cap", [(200_000, 7680, 4320, 3_000_000), (300_000, 7680, 4320, 3_000_000),
                                       (1_000_000, 7680, 4320, 3_000_000), (1_000_000, 7680, 4320, 5_000_000),
                                       (1_000_000, 5120, 2880, 5_000_000), (20_000, 16384, 16384, 5_200_000),
                                       (1_000_000, 16384, 16384, 4_500_000)])
def test_static_scratch_keeps_the_gpu_busy(plan, n, w, h, cap):
    (nbytes, chunks, _), (_, free, _) = plan([(1, n, w, h, cap, STATIC), (1, n, w, h, cap, 0)])
    assert nbytes <= STATIC
    # half the chunks that no limit would give, at least: one halving leaves 128 workgroups
    assert chunks >= (free + 1) // 2
    assert _groups(1, n, w, h, chunks) >= min(100, n // 2048)


def test_static_scratch_is_enough_whenever_it_was(plan):
    """Every call whose stated size fits the scratch has a layout that fits; the others stay refused."""
    rng = np.random.default_rng(3)
    calls = []
    for _ in range(3000):
        nv = int(rng.integers(1, 4)) if rng.uniform() < 0.8 else int(2 ** rng.uniform(0, 12))
        w, h = (int(2 ** rng.uniform(0, 15)) for _ in range(2))
        calls.append((nv, min(int(2 ** rng.uniform(0, 25)), (2 ** 31 - 1) // nv), w, h, int(2 ** rng.uniform(0, 22.9)), STATIC))
    told = np.array([_told(*c[:5]) for c in calls])
    got = plan(calls)[:, 0]
    assert 500 < (told <= STATIC).sum() < 2900
    np.testing.assert_array_equal(got <= STATIC, told <= STATIC)


def test_memory_is_bounded_however_many_tiles(plan):
    """20 bytes per entry and tile as stated, or 12 per entry, 8 per particle, 16 per tile and the
    matrix: 512 rows of 36864 counts at most (75 MB) and a row per view."""
    calls = [(nv, n, w, h, cap, 0) for nv in (1, 3, 20) for n in (5000, 1_000_000, 6_000_000)
             for w, h in ((1920, 1080), (3840, 2160), (7680, 4320), (12288, 6912), (16384, 16384), (32768, 32768))
             for cap in (1_000_000, 5_000_000, 50_000_000)]
    for c, (nbytes, chunks, boxes) in zip(calls, plan(calls)):
        nv, n, w, h, cap, _ = c
        tiles = nv * _tiles(w, h)
        matrix = 4 * (512 * BAND + tiles)
        assert boxes and nbytes <= max(_told(nv, n, w, h, cap), 12.6 * cap + 8 * nv * n + 16 * tiles + matrix + (1 << 20)), c
        # (the single rows of 20 small shares are at most twice that many workgroups)
        assert _groups(*c[:4], chunks) <= 2 * 512 + nv * -(-_tiles(w, h) // BAND), c
