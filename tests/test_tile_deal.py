"""The choice of how the blend launches deal their tiles to the XCDs (CPU: the
host side of common.h's functions, compiled here).  Eight workgroups make the
choice, each for itself; the launch takes every tile once only if all make the
same one.  So the choice may not depend on the order in which partial sums are
added, and every chunking is a bijection."""
import ctypes as C
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

HARNESS = r"""
#include "common.h"
using namespace xg;
// the choice with every (step, XCD) load's shares added in the order order[]
extern "C" int choose(const uint32_t *group, int n, int g, const int32_t *order) {
    std::remove_cv_t<std::remove_reference_t<decltype(deal_share(group, g, TileDeal(n, n, true), 0, 0))>> zero = 0;
    float excess[kDealSteps];
    for (int s = 0; s < kDealSteps; ++s) {
        decltype(zero) largest = zero, total = zero;
        for (int x = 0; x < kXcds; ++x) {
            const TileDeal d(n, deal_chunk(n, g, s), s == 0);
            decltype(zero) load = zero;
            for (int p = 0; p < kDealParts; ++p)
                load += deal_share(group, g, d, x, order[(s * kXcds + x) * kDealParts + p]);
            largest = load > largest ? load : largest;
            total += load;
        }
        excess[s] = deal_excess(largest, total);
    }
    return deal_choice(excess);
}
extern "C" int words() { return kDealSteps * kXcds * kDealParts; }
// the tiles in launch order under step s
extern "C" void tiles(int n, int g, int s, int32_t *out) {
    const TileDeal d(n, deal_chunk(n, g, s), s == 0);
    for (int x = 0; x < kXcds; ++x)
        for (int j = 0; j < d.tiles(x); ++j) *out++ = d.tile(x, j);
}
extern "C" void sample(int ng, int g, int64_t *out) {
    for (int k = 0; k < ng; ++k)
        for (int l = 0; l < 16; ++l) *out++ = order_sample(k, l, g);
}
extern "C" int groups() { return kOrderGroups; }
// the loads
extern "C" void loads(const uint32_t *group, int n, int g, double *out) {
    for (int s = 0; s < kDealSteps; ++s)
        for (int x = 0; x < kXcds; ++x) {
            const TileDeal d(n, deal_chunk(n, g, s), s == 0);
            double sum = 0;
            for (int p = 0; p < kDealParts; ++p) sum += (double)deal_share(group, g, d, x, p);
            *out++ = sum;
        }
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    if not os.path.exists(HIPCC) and not shutil.which(HIPCC):
        pytest.skip("hipcc not installed")
    d = tmp_path_factory.mktemp("deal")
    src, so = str(d / "deal.cpp"), str(d / "libdeal.so")
    with open(src, "w") as f:
        f.write(HARNESS)
    subprocess.check_call([HIPCC, "-x", "hip", "--offload-host-only", "-O2", "-std=c++17", "-fPIC", "-shared",
                           f"-I{ROOT}/include", f"-I{ROOT}/paper_2403_04116_amd/csrc", "-include", "type_traits", src, "-o", so])
    return C.CDLL(so)


def _ptr(a):
    return a.ctypes.data_as(C.c_void_p)


def _group_tiles(n):
    g = 16
    while -(-n // g) > 2048:
        g *= 2
    return g


def _one_choice(lib, group, n, g, rng):
    picks = set()
    for _ in range(24):
        order = np.concatenate([rng.permutation(8) for _ in range(lib.words() // 8)]).astype(np.int32)
        picks.add(lib.choose(_ptr(group), n, g, _ptr(order)))
    assert len(picks) == 1, (n, picks)


@pytest.mark.parametrize("n", [1023, 12_294, 102_400])
@pytest.mark.parametrize("mean", [60, 20_000])
def test_one_choice_for_repeating_views(lib, n, mean):
    # equal loads under several chunkings
    rng = np.random.default_rng(n + mean)
    g = _group_tiles(n)
    ng = -(-n // g)
    for _ in range(8):
        wave = rng.integers(0, 2 * mean * g, int(rng.integers(2, max(3, ng // 8))))
        _one_choice(lib, np.tile(wave, ng)[:ng].astype(np.uint32), n, g, rng)


@pytest.mark.parametrize("seed", range(60))
def test_one_choice_for_a_heavy_last_view(lib, seed):
    # the entries in the left-over piece: loads of the finer chunkings differ
    # by roundings only (float shares disagree in 8 of these 60 frames)
    rng = np.random.default_rng(seed)
    n = int(rng.integers(2000, 60000))
    g = _group_tiles(n)
    ng = -(-n // g)
    group = rng.integers(0, 20, ng)
    k = int(rng.integers(1, 40))
    group[-k:] = rng.integers(0, 20_000_000, k)
    _one_choice(lib, group.astype(np.uint32), n, g, np.random.default_rng(seed + 1))


@pytest.mark.parametrize("n", [1, 7, 8, 9, 100, 1023, 1024, 4099, 40_003, 262_147])
def test_every_chunking_is_a_bijection(lib, n):
    g = _group_tiles(n)
    for step in range(7):
        out = np.full(n, -1, np.int32)
        lib.tiles(n, g, step, _ptr(out))
        np.testing.assert_array_equal(np.sort(out), np.arange(n))


def test_choice_takes_an_even_split(lib):
    # even frames stay contiguous; one heavy eighth is dealt out
    n, g = 8192, 16
    order = np.tile(np.arange(8), lib.words() // 8).astype(np.int32)
    assert lib.choose(_ptr(np.full(n // g, 500, np.uint32)), n, g, _ptr(order)) == 0
    heavy = np.full(n // g, 10, np.uint32)
    heavy[:n // g // 8] = 5000
    loads = np.zeros((7, 8))
    lib.loads(_ptr(heavy), n, g, _ptr(loads))
    assert loads[0].max() > 7.0 * loads[0].mean()
    best = lib.choose(_ptr(heavy), n, g, _ptr(order))
    assert best > 0 and loads[best].max() <= 1.1 * loads[best].mean()


@pytest.mark.parametrize("n", [1, 100, 32_768, 32_769, 262_147, 1_024_000, 1 << 27])
def test_order_reads_a_bounded_number_of_tiles(lib, n):
    g = _group_tiles(n)
    ng = -(-n // g)
    assert ng <= lib.groups() == 2048
    out = np.zeros(16 * ng, np.int64)
    lib.sample(ng, g, _ptr(out))
    # one tile of every stretch of g / 16: at most 32 768, every tile of small frames
    np.testing.assert_array_equal(out // (g // 16), np.arange(16 * ng))
    if n <= 32_768:
        np.testing.assert_array_equal(out, np.arange(16 * ng))
    elif g >= 512:      # no column of 32 taken more than twice as often as its share
        assert np.bincount(out % 32, minlength=32).max() < 2 * out.size / 32


def _sampled_choice(lib, lens):
    n = lens.size
    g = _group_tiles(n)
    ng = -(-n // g)
    t = np.zeros(16 * ng, np.int64)
    lib.sample(ng, g, _ptr(t))
    group = np.where(t < n, lens[np.minimum(t, n - 1)], 0).reshape(ng, 16).sum(1).astype(np.uint32)
    order = np.tile(np.arange(8), lib.words() // 8).astype(np.int32)
    return lib.choose(_ptr(group), n, g, _ptr(order)), g


def test_choice_from_the_sample(lib):
    y, x = np.mgrid[-1:1:32j, -1:1:32j]
    view = (40 * np.exp(-3 * (x * x + y * y))).astype(np.int64).ravel()      # 512 x 512, centre heavy
    assert _sampled_choice(lib, np.tile(view, 1000))[0] == 0                   # equal views: contiguous
    lens = np.concatenate([np.tile(view, 400), np.full(600 * 16, 300)])        # small views last, long lists
    best, g = _sampled_choice(lib, lens)
    assert best > 0
    out = np.zeros(lens.size, np.int32)
    lib.tiles(lens.size, g, best, _ptr(out))
    split = [c.sum() for c in np.array_split(lens[out], 8)]
    whole = [c.sum() for c in np.array_split(lens, 8)]
    assert max(whole) > 1.3 * np.mean(whole) and max(split) < 1.15 * np.mean(split)
