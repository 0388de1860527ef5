#ifndef SL_UNIT_PLAN_H
#define SL_UNIT_PLAN_H
// The host's plan of a one-launch step (engine.cpp): how many workgroups each
// unit of a step gets, or that the step should take two launches.
#include <algorithm>

#include "engine_internal.h"

namespace sl {

// One-launch step: taken only while its longest wave range is within
// kUnitSlackTiles tiles of a split-kernel worker's share (the two-launch
// step spreads tiles over all workers but pays a second launch).
constexpr int kUnitSlackTiles = 8;
// What merging a unit's pieces costs, in tiles of a wave's stream: once the
// unit has more than one workgroup, and again per eight workgroups more.
// Generations with kMergeTiles / kMergeMoreTiles of 2 / 1, 4 / 1, 2 / 2, 4 / 2
// and 5 / 2 (MI355X, ms; without the rule 30.2, 27.1, 4.6 and 36.4):
//   96 samples on 32 slots, bf16        30.1   30.0   29.3   29.1   29.4
//   the same, E4M3                      26.7   26.7   25.5   25.2   25.3
//   2 short samples on one slot, bf16    4.5    4.3    4.6    4.2    4.2
//   32 samples on 24 slots, 64/8 heads  36.2   36.2   33.7   33.7   33.7
constexpr int kMergeTiles = 4;
constexpr int kMergeMoreTiles = 2;
// What workgroups beyond the chip's first pass cost, in the same tiles: they
// start late (46 sequences x 4 KV heads, a fifth of them long, E4M3: 304
// workgroups with waves of 5 tiles 13.2 us a step, 224 with 9 12.7).
constexpr int kSecondPassTiles = 6;

// The most a wave streams in a plan that does not fit the chip in one pass:
// with more, waves that end unevenly cost more than a second launch (122
// sequences x 2 KV heads, a fifth of them long, bf16 with head_dim 128, waves of
// 11 tiles = 88 KB: 40.7 us a step, 36.7 in two launches; 25 x 8, head_dim 64,
// 51 tiles = 204 KB: 87 and 70; 49 x 4, head_dim 64, 15 tiles = 60 KB: 24.6 and 28.8).
constexpr int kSecondPassBytes = 64 << 10;

inline int merge_cost(int k) { return (k > 1 ? kMergeTiles : 0) + (k - 1) / 8 * kMergeMoreTiles; }

// A unit's workgroups and shares (UnitStepParams::split): its `nb` tiles over
// `k` workgroups.
inline uint32_t unit_split(int nb, int k)
{
    const int waves = k * kUnitWaves;
    return (uint32_t)(k - 1) | (uint32_t)(nb % waves) << 6 | (uint32_t)(nb / waves) << 16;
}

// The fewest workgroups that leave a wave of a unit of nb tiles at most `share`
// (below 2^16).
inline int groups_of(int nb, int share)
{
    const unsigned per = (unsigned)(kUnitWaves * share);
    return (unsigned)nb <= per ? 1 : (int)(((unsigned)nb + per - 1) / per);
}

// Tiles per wave of the plan whose workgroups fit the chip in one pass, the
// longest wave of which sets the stream's time: the smallest (to a sixteenth),
// or one that saves as much merging; 0 if it would be more than `most`.
// (Giving every unit the whole part of its share of the CUs left some waves
// with nearly twice the tiles of others: a 96-sample generation took 33.2
// instead of 32.5 ms.)
inline int one_pass_share(const int32_t *len, int n, int num_kv_heads, int cus, long long tiles, int longest, int most)
{
    // Whether the workgroups fit the chip; more tiles per wave never need more.
    auto fits = [&](int wave_tiles) {
        if (groups_of(longest, wave_tiles) > kMaxUnitSplit)
            return false;
        int blocks = 0;
        for (int e = 0; e < n && blocks <= cus; ++e)
            blocks += num_kv_heads * groups_of((len[e] + kPageSize - 1) / kPageSize, wave_tiles);
        return blocks <= cus;
    };
    // (Trying one share after the other, up to the one that fitted, took 34 us
    // of host time per step for 128 sequences, one of them long; now 0.2.)
    const long long all_waves = (long long)cus * kUnitWaves;
    int wave_tiles = (int)std::max(1LL, (tiles * num_kv_heads + all_waves - 1) / all_waves);
    if (wave_tiles > most)
        return 0;
    int lo = wave_tiles, hi = wave_tiles;
    if (!fits(lo)) {   // (most small steps fit at once)
        if (!fits(most))
            return 0;
        ++lo;
        hi = most;
    }
    while (lo < hi) {   // hi fits
        const int mid = lo + (hi - lo) / 2;
        if (fits(mid))
            hi = mid;
        else
            lo = mid + 1;
    }
    while (wave_tiles < hi)
        wave_tiles += std::max(1, wave_tiles / 16);
    if (wave_tiles > most)
        return 0;
    // Fewer and longer shares can still be faster, as the pieces of a unit cost
    // a merge: the units in at most eight workgroups each (one batch of loads
    // for whoever merges them), or in one (no merge).
    auto cost = [longest](int w) { return w + merge_cost(groups_of(longest, w)); };
    int best = wave_tiles;
    for (const int k : {8, 1}) {
        const int w = (longest + kUnitWaves * k - 1) / (kUnitWaves * k);
        if (w > wave_tiles && w <= most && cost(w) < cost(best))
            best = w;
    }
    return best;
}

// Plan n sequences (len[e] >= 1) with num_kv_heads units each on `cus` CUs;
// `workers` is the two-launch step's worker count, tile_bytes what a wave reads
// per tile (K and V). Fills first[0 .. n] and
// split[0 .. n) (UnitStepParams) and returns the workgroups, or 0 for two
// launches.
//
// The units get the fewest workgroups that leave every wave at most
// one_pass_share tiles. With a few long sequences among so many short ones that
// their units, a workgroup each, fill most of the chip, there is no such plan,
// or its longest wave has far more than the mean. Every unit then gets the
// whole part of its share of the CUs, as long as the workgroups too many start
// when the short ones end, within kSecondPassBytes and with the longest wave
// near the mean (a second launch counted as kUnitSlackTiles, and the rounds a
// quarter longer than their waves say). Per step, MI355X, in one pass or two
// launches -> with such a plan:
//   128 sequences x 2 KV heads, 32000 and 200.. tokens     28.7 -> 20.9 us; E4M3 26.7 -> 16.2
//   54 x 4, one to three of 32000, the others short, E4M3  31.8 -> 26.4
//   53 x 4, lognormal up to 40000                           148 -> 129
inline int plan_units(const int32_t *len, int n, int num_kv_heads, int cus, int workers, int tile_bytes,
                      int32_t *first, uint32_t *split)
{
    if (n == 0 || (long long)n * num_kv_heads > cus)
        return 0;
    int longest = 0;
    long long tiles = 0;   // per KV head
    for (int e = 0; e < n; ++e) {
        const int nb = (len[e] + kPageSize - 1) / kPageSize;
        tiles += nb;
        longest = std::max(longest, nb);
    }
    const long long worker_tiles = (tiles * num_kv_heads + workers - 1) / workers;
    const int most = std::min((int)worker_tiles + kUnitSlackTiles, (1 << 16) - 1);   // (the quotients' field)
    const int share = one_pass_share(len, n, num_kv_heads, cus, tiles, longest, most);
    auto place = [&](auto groups) {   // groups(nb): the workgroups of a unit of nb tiles
        int blocks = 0;
        for (int e = 0; e < n; ++e) {
            const int nb = (len[e] + kPageSize - 1) / kPageSize, k = groups(nb);
            first[e] = blocks;
            split[e] = unit_split(nb, k);
            blocks += num_kv_heads * k;
        }
        return first[n] = blocks;
    };
    const long long all_waves = (long long)cus * kUnitWaves;
    if (share == 0 || (share > kSecondPassTiles + 1 && share * all_waves > 2 * tiles * num_kv_heads)) {
        int wave = 0, most_groups = 1, long_blocks = 0;
        const int blocks = place([&](int nb) {
            const int whole = (int)std::min((long long)cus * nb / (tiles * num_kv_heads), (long long)kMaxUnitSplit);
            const int k = std::max(1, std::min(whole, (nb + kUnitWaves - 1) / kUnitWaves));
            wave = std::max(wave, (nb + kUnitWaves * k - 1) / (kUnitWaves * k));
            most_groups = std::max(most_groups, k);
            return k;
        });
        if (wave >= 1 << 16)
            return 0;
        for (int e = 0; e < n; ++e)   // those with more than half of the longest wave
            if (2 * (int)(split[e] >> 16) >= wave)
                long_blocks += first[e + 1] - first[e];
        const long long rounds = (long long)wave * std::max(1, (long_blocks + cus - 1) / cus);
        if (share == 0)
            return rounds * tile_bytes <= kSecondPassBytes &&
                           5 * rounds * all_waves <= 4 * (tiles * num_kv_heads + kUnitSlackTiles * all_waves)
                       ? blocks
                       : 0;
        if (rounds + merge_cost(most_groups) + (blocks > cus ? kSecondPassTiles : 0) <
            share + merge_cost(groups_of(longest, share)))
            return blocks;
    }
    return place([share](int nb) { return groups_of(nb, share); });
}

}  // namespace sl

#endif  // SL_UNIT_PLAN_H
