"""The engine's host plan of a one-launch step (CPU only), compiled for the host: the rule against a
plain statement of it, its cost, and which of the kernel's merge branches the GPU tests' batches reach."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from paper_2504_15930_amd import build

CUS = 256   # of an MI355X, and four (three for bf16 with head_dim 128) workers per CU
# Steps of the GPU tests of merged units: pages per sequence, KV heads, workgroups of the longest unit.
# One workgroup writes the rows; up to eight pieces are merged in one batch of loads, more in batches
# of eight; and more workgroups than CUs.
MERGED = {"one": ([1, 8, 3], 2, 1), "seven": ([200], 2, 7), "eight": ([300], 1, 8), "nine": ([1152] * 3, 9, 9),
          "sixteen": ([512] * 2, 8, 16), "seventeen": ([544] * 2, 7, 17), "thirty-two": ([768], 1, 32),
          "past the chip": ([500] + [12] * 127, 2, 31)}
LONG_PROMPT = 11000   # tokens of the long sample among short ones, in more than eight workgroups

SOURCE = r"""
#include <chrono>
#include <vector>
#include "unit_plan.h"
using namespace sl;
// The rule, stated plainly: every share from the smallest one up.
static int stepped(const int32_t *len, int n, int hkv, int cus, int workers, int bytes, int32_t *first, uint32_t *split)
{
    if (n == 0 || (long long)n * hkv > cus)
        return 0;
    long long tiles = 0;
    int longest = 0;
    for (int e = 0; e < n; ++e) {
        tiles += (len[e] + 15) / 16;
        longest = std::max(longest, (len[e] + 15) / 16);
    }
    auto plan = [&](int share) {
        const int per = kUnitWaves * share;
        int blocks = 0;
        for (int e = 0; e < n; ++e) {
            const int nb = (len[e] + 15) / 16, k = (nb + per - 1) / per, waves = k * kUnitWaves;
            if (k > kMaxUnitSplit)
                return cus + 1;
            first[e] = blocks;
            split[e] = (uint32_t)(k - 1) | (uint32_t)(nb % waves) << 6 | (uint32_t)(nb / waves) << 16;
            blocks += hkv * k;
        }
        first[n] = blocks;
        return blocks;
    };
    const long long waves = (long long)cus * kUnitWaves, worker = (tiles * hkv + workers - 1) / workers;
    int share = (int)std::max(1LL, (tiles * hkv + waves - 1) / waves), blocks;
    while ((blocks = plan(share)) > cus)
        share += std::max(1, share / 16);
    auto cost = [&](int w) {
        const int k = (longest + kUnitWaves * w - 1) / (kUnitWaves * w);
        return w + (k > 1 ? kMergeTiles : 0) + (k - 1) / 8 * kMergeMoreTiles;
    };
    int best = share;
    for (int k : {8, 1}) {
        const int w = (longest + kUnitWaves * k - 1) / (kUnitWaves * k);
        if (w > share && w <= worker + kUnitSlackTiles && cost(w) < cost(best))
            best = w;
    }
    if (best != share)
        blocks = plan(share = best);
    const bool one_pass = share < 1 << 16 && share <= worker + kUnitSlackTiles;
    // The whole part of every unit's share of the CUs instead: where one pass is refused and this
    // takes little more than the mean, or where one pass leaves the longest wave more than twice
    // the mean and more than this does.
    if (one_pass && (share <= kSecondPassTiles + 1 || (double)share <= 2.0 * tiles * hkv / waves))
        return blocks;
    std::vector<int> ks(n), least(n);
    int wave = 0, most_k = 1, total = 0, longer = 0;
    for (int e = 0; e < n; ++e) {
        const int nb = (len[e] + 15) / 16;
        ks[e] = (int)std::max(1LL, std::min({(long long)cus * nb / (tiles * hkv), (nb + 7LL) / 8, 32LL}));
        least[e] = nb / (8 * ks[e]);
        wave = std::max(wave, (nb + 8 * ks[e] - 1) / (8 * ks[e]));
        most_k = std::max(most_k, ks[e]);
        total += hkv * ks[e];
    }
    if (wave >= 1 << 16)
        return 0;
    for (int e = 0; e < n; ++e)
        longer += 2 * least[e] >= wave ? hkv * ks[e] : 0;
    const double rounds = (double)wave * std::max(1, (longer + cus - 1) / cus);
    auto merging = [](int k) { return (k > 1 ? kMergeTiles : 0) + (k - 1) / 8 * kMergeMoreTiles; };
    const int late = total > cus ? kSecondPassTiles : 0;
    if (one_pass ? rounds + merging(most_k) + late >= cost(share)
                 : rounds * bytes > kSecondPassBytes || 1.25 * rounds > (double)tiles * hkv / waves + kUnitSlackTiles)
        return one_pass ? blocks : 0;
    total = 0;
    for (int e = 0; e < n; ++e) {
        const int nb = (len[e] + 15) / 16, k = ks[e];
        first[e] = total;
        split[e] = (uint32_t)(k - 1) | (uint32_t)(nb % (8 * k)) << 6 | (uint32_t)(nb / (8 * k)) << 16;
        total += hkv * k;
    }
    return first[n] = total;
}
extern "C" int plan(int plain, const int32_t *len, int n, int hkv, int cus, int workers, int bytes, int32_t *first,
                    uint32_t *split)
{
    return (plain ? stepped : plan_units)(len, n, hkv, cus, workers, bytes, first, split);
}
extern "C" double microseconds(int plain, const int32_t *len, int n, int hkv, int cus, int workers, int bytes)
{
    std::vector<int32_t> first(n + 1);
    std::vector<uint32_t> split(n);
    double best = 1e30;
    for (int r = 0; r < 20; ++r) {
        const auto t0 = std::chrono::steady_clock::now();
        for (int i = 0; i < 100; ++i)
            plan(plain, len, n, hkv, cus, workers, bytes, first.data(), split.data());
        best = std::min(best, std::chrono::duration<double, std::micro>(std::chrono::steady_clock::now() - t0).count() / 100);
    }
    return best;
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "plan.cpp").write_text(SOURCE)
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    out = str(d / "plan.so")
    subprocess.run(["g++", "-std=c++17", "-O2", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__", "-I",
                    os.path.join(rocm, "include"), "-I", build.CSRC, str(d / "plan.cpp"), "-o", out], check=True)
    lib = ctypes.CDLL(out)
    lib.microseconds.restype = ctypes.c_double
    return lib


def _plan(lib, lens, hkv, workers, cus=CUS, plain=False, tile=8192):
    """(workgroups, first, split) of a step, or None for two launches."""
    lens = np.ascontiguousarray(lens, np.int32)
    first, split = np.full(len(lens) + 1, -1, np.int32), np.zeros(len(lens), np.uint32)
    p = [a.ctypes.data_as(ctypes.c_void_p) for a in (lens, first, split)]
    blocks = lib.plan(int(plain), p[0], len(lens), hkv, cus, workers, tile, p[1], p[2])
    return (blocks, first.tolist(), split.tolist()) if blocks else None


@pytest.mark.parametrize("seed", range(6))
def test_plan_is_the_rule(lib, seed):
    rng = np.random.default_rng(seed)
    one = 0
    for _ in range(600):
        hkv = int(rng.choice([1, 2, 3, 4, 8, 12]))
        cus = int(rng.choice([256, 256, 64, 304]))
        n = int(rng.integers(1, max(2, min(128, cus // hkv + 2))))
        lens = rng.integers(1, int(rng.choice([17, 300, 5000, 60000])), n)
        if rng.random() < .5:
            lens[rng.integers(0, n)] = int(rng.integers(1, 500000))
        workers = int(rng.choice([768, 1024, 1, 100, 4096]))
        tile = int(rng.choice([2048, 4096, 8192]))
        got, want = (_plan(lib, lens, hkv, workers, cus, plain, tile) for plain in (False, True))
        assert got == want, (hkv, cus, workers, lens.tolist())
        one += got is not None
    assert one > 100


def test_plan_covers_every_unit(lib):
    """The workgroups of a plan: in order, at most two for each CU, and their waves' shares add up to
    the unit's pages."""
    rng = np.random.default_rng(9)
    for _ in range(600):
        lens = rng.integers(1, 9000, rng.integers(1, 60))
        if rng.random() < .5:
            lens = lens // 50 + 1
            lens[0] = rng.integers(1, 100000)
        got = _plan(lib, lens, 4, 768)
        if got is None:
            continue
        blocks, first, split = got
        assert first[0] == 0 and first[-1] == blocks <= 2 * CUS
        for e, L in enumerate(lens):
            k, rem, per = (split[e] & 63) + 1, split[e] >> 6 & 1023, split[e] >> 16
            assert first[e + 1] - first[e] == 4 * k and k <= 32 and rem < 8 * k
            assert per * 8 * k + rem == -(-int(L) // 16)


@pytest.mark.parametrize("workers,tile", [(768, 8192), (1024, 2048)])
@pytest.mark.parametrize("name", MERGED)
def test_batches_that_reach_every_merge(lib, name, workers, tile):
    pages, hkv, groups = MERGED[name]
    blocks, _, split = _plan(lib, [16 * n - 4 for n in pages], hkv, workers, tile=tile)
    assert max((s & 63) + 1 for s in split) == groups
    assert (blocks > CUS) == (name == "past the chip")


@pytest.mark.parametrize("workers,hkv", [(768, 2), (1024, 2), (1024, 1)])
def test_a_long_prompt_among_short_ones_is_merged_in_batches(lib, workers, hkv):
    _, _, split = _plan(lib, [LONG_PROMPT + 1] + [300] * 15, hkv, workers)
    assert (split[0] & 63) + 1 > 16


@pytest.mark.parametrize("lens,hkv", [([2**31 - 16], 1), ([2**28, 2**27], 4)])
def test_shares_past_the_quotients_field_take_two_launches(lib, lens, hkv):
    assert _plan(lib, lens, hkv, 1) is None and _plan(lib, lens, hkv, 1, plain=True) is None


def test_one_long_sequence_among_many_short_ones_takes_one_launch(lib):
    """Also where the units, a workgroup each, fill the chip: two launches were slower."""
    for lens, hkv in (([32000] + [200] * 127, 2), ([16000] + [100] * 63, 4)):
        for workers in (768, 1024):
            blocks, first, split = _plan(lib, lens, hkv, workers)
            assert blocks > CUS and (split[0] & 63) == 31


def test_plan_of_one_long_sequence_among_many_costs_little(lib):
    """Trying share after share costs many times the plan's passes."""
    lens = np.array([32000] + [200] * 127, np.int32)
    p = lens.ctypes.data_as(ctypes.c_void_p)
    ours, plain = (lib.microseconds(v, p, len(lens), 2, CUS, 768, 8192) for v in (0, 1))
    assert ours < plain / 5, (ours, plain)
