// Internal interface between the host-side entry points (api.cpp) and the
// gfx950 kernels (decode_split.hip and decode_shared.hip with the worker in
// decode_unit.h; append.hip and merge.hip with the append worker in
// append_unit.h; engine.hip), and the decode engine (engine.cpp).
//
// Work decomposition. A "unit" is one (sequence b, KV head g) pair and owns
// n_b = ceil(L_b / 16) page-head tiles (16 tokens x head_dim of one KV head).
// A step is NT = 1, 2 or 4 consecutive tiles of a unit (step_tiles in
// decode_unit.h; fewer at the unit's end). Units are laid out b-major, g-minor,
// and their steps are numbered consecutively, giving W = Hkv * sum_b
// ceil(n_b / NT) steps in total. Worker w (one wavefront) owns steps
// [floor(w W / NW), floor((w + 1) W / NW)): every worker takes the same number
// of steps (+-1) whatever the length skew, so a few very long sequences are
// spread over many workers instead of leaving most of the chip idle (the
// on-chip analogue of StreamRL's skewness bubbles, Section 2.4 and Section
// 5.1). In tiles the ranges are as equal as the units' last steps are full: a
// range of sequences of one page has 1 / NT of the tiles of one in a long
// sequence.
//
// A worker streams its range as one flat sequence of steps, which every
// workgroup derives itself: it scans the lengths (and, with prefix sharing,
// the group descriptions) into LDS, and every wavefront works out its range 64
// steps at a time, one per lane: the unit by binary search, the pages, and
// their block-table entries, loaded while the 64 steps before stream. There is
// no partitioning launch and no list of steps in memory, and unit boundaries
// inside the range cost no dependent load and do not drain the load pipeline.
//
// (For the shared pages of prefix-shared attention a worker is a workgroup
// whose four wavefronts stream the same range, one query block each.)
//
// A unit that lies inside one worker's range is finished by that worker; a
// unit cut by a range boundary leaves one partial softmax state per worker
// that touched it, combined afterwards by the merge kernel. Worker w writes
// the piece its range starts with to slot 2w and, if its range ends inside a
// later unit, that trailing piece to slot 2w + 1.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <hip/hip_runtime.h>

namespace sl {

constexpr int kPageSize = 16;
constexpr int kWave = 64;
constexpr int kWavesPerBlock = 4;          // split kernel: 4 independent workers per block
constexpr int kMaxGroup = 16;              // query heads per KV head (one MFMA column block)
constexpr int kMaxBatch = 8192;            // the split kernel keeps two ints per sequence in LDS
constexpr int kMergeThreads = 256;         // one wave per (sequence, query head)
constexpr int kMaxWorkers = 1 << 16;       // keeps partial-state offsets below 2^31 bytes
// A worker is given at least this many tiles: a small stream (a small batch, a
// short context) is split over fewer workers rather than cut into pieces of
// one or two tiles, each of which would cost a partial state and a merge step.
// Calls with eight -> four tiles (MI355X, kernels and the gap between them):
//   8 sequences of 1..256 tokens, D = 64        10.2 -> 8.2 us
//   one sequence of 512, 28/4 heads              9.9 -> 8.4
//   64 of 1..200, 28/4 heads                    15.5 -> 12.2
//   256 of 1..120, 28/4 heads                   20.2 -> 18.5
//   3 prompts x 22 samples of ~23 own tokens    25.0 -> 21.5
// With two, 8 prompts x 8 samples of ~60 own tokens took 26.5 instead of 21.7.
constexpr int kMinTiles = 4;
// E4M3: a tile is half as long, and a piece costs as much, so beyond half of
// the workers it takes this many (64 of 1..200 tokens, below it, 12.6 -> 10.4
// us with four; 256 of 1..120, beyond it, 14.4 -> 15.4). The shared units of
// prefix sharing, whose pieces have kPrefixRows rows, take this many always
// (with four, 3 prompts x 16 samples, 12 heads, D = 64, 26.7 -> 28.6).
constexpr int kMinTilesWide = 8;

// Workers that take part in a stream of `total` steps of step_tiles tiles (the
// others exit at once); both the split kernel and the merge derive it from the
// same total. A unit's last step counts as a full one (below 2^30 tiles so
// counted). `wide`: kMinTilesWide beyond this many workers.
__host__ __device__ inline int effective_workers(long long total, int num_workers, int step_tiles, int wide)
{
    const int tiles = (int)total * step_tiles;
    const int few = (tiles + kMinTilesWide - 1) / kMinTilesWide;
    int want = (tiles + kMinTiles - 1) / kMinTiles;
    want = want < wide ? want : wide;
    want = want > few ? want : few;
    return want < 1 ? 1 : (want < num_workers ? want : num_workers);
}
// `wide` for plain attention's stream and the own pages of prefix sharing; the
// shared pages' is 0.
__host__ __device__ inline int wide_from(int num_workers, bool fp8) { return fp8 ? num_workers / 2 : num_workers; }
// Prefix sharing: shared-page workgroups that take part in a call. The launch
// holds the own-page workgroups and up to twice `base` shared ones, and a CU
// holds two such workgroups; own-page workgroups without work exit at once,
// and shared workgroups beyond `base` take their slots, so that a batch with
// few own pages still streams its shared pages with two workgroups per CU. All
// ranges are equally long, and on a CU with two shared workgroups each takes
// longer: with few such CUs their ranges end late, so beyond `base` there are
// three quarters of it or none. Shared workgroups (base 256) and time, MI355X:
//   130 prompts of 7030 tokens x 14 samples, 16/1 heads, D = 128   284 619 us, 256 493
//   32 of 4000 x 16, 28/4 heads                                    382 169 us, 256 148
//   32 of 4000 x 16, 16/1 heads                                    480  76 us, 256  83
// The split kernel and the merge derive it from the same totals (own tiles).
__host__ __device__ inline int effective_shared_workers(long long own_total, int own_workers, int base,
                                                        int max_workers, int step_tiles, bool fp8)
{
    const int own_blocks = (own_workers + kWavesPerBlock - 1) / kWavesPerBlock;
    const int active =
        own_total > 0
            ? (effective_workers(own_total, own_workers, step_tiles, wide_from(own_workers, fp8)) + kWavesPerBlock - 1) /
                  kWavesPerBlock
            : 0;
    const int idle = own_blocks - active;
    const int n = 4 * idle >= 3 * base ? base + (idle < base ? idle : base) : base;
    return n < max_workers ? n : max_workers;
}
constexpr size_t kAlign = 256;

// ceil(2^32 / group) (2^32 itself, for a group of 1, does not fit): h / group
// is the high half of h times this, exact for h group < 2^32.
inline uint32_t inverse_of(int group) { return (uint32_t)(((1ull << 32) + (unsigned)group - 1) / (unsigned)group); }

// Step metadata, one word per step of a stream:
//   [4] last step of its unit, [5] first step of its unit, [6] the sequence
//   length is invalid or the block table named a page outside the pool,
//   [7] see kMetaPrefixed, [31:8] the unit, b * Hkv + g (its first query row
//   over G).
// A tile's KV data is page-head tile page_id * Hkv + g of the
// [num_pages][Hkv] grid.
constexpr uint32_t kMetaLast = 1u << 4;
constexpr uint32_t kMetaFirst = 1u << 5;
constexpr uint32_t kMetaBad = 1u << 6;
constexpr uint32_t kMetaPrefixed = 1u << 7;   // own-page unit of a sequence whose first pages are shared
// Prefix-sharing mode: the shared-page stream holds, per (group, KV head),
// the group's shared pages once (every shared page is full); their metadata
// names the unit of the group's first member. The query rows of a shared unit are (member j, head h) ->
// row0 + j * Hq + h, at most kPrefixRows of them (kPrefixBlocks MFMA column
// blocks of 16).
constexpr int kPrefixBlocks = 4;
constexpr int kPrefixRows = 16 * kPrefixBlocks;
constexpr int kMetaUnitShift = 8;

struct Workspace {
    int32_t *cum_pages;   // [B + 1] exclusive prefix sum of steps per sequence and KV head (written by the split kernel)
    float *part_ml;       // [2 NW][G][2]  (running max in log2 units, sum of weights)
    float *part_acc;      // [2 NW][G][D]  un-normalised weighted value sums
};

struct SplitParams {
    const uint16_t *q;
    const void *k_pages;
    const void *v_pages;
    const float *k_scales;
    const float *v_scales;
    uint16_t *out;
    float *part_ml;
    float *part_acc;
    int32_t batch, num_kv_heads, group, num_workers;
    int32_t num_q_heads;   // query-row stride of one sequence (prefix mode)
    float scale_log2;      // scale * log2(e): scores are kept in base-2 units
    // Prefix mode: a unit seen whole by one worker that still has to be merged
    // (a shared unit, or the own pages of a sequence with shared pages) keeps
    // its partial state here, at unit index (first query row) / G, with the
    // row stride of part_ml / part_acc; null otherwise.
    float *unit_ml;
    float *unit_acc;
    // The kernel derives every tile from the lengths and the block table
    // itself; workgroup 0 stores the prefix sum of steps in cum_out for the merge
    // (plain attention; prefix sharing stores its sums through PrefixParams).
    const int32_t *seq_lens;
    const int32_t *block_table;
    int32_t *cum_out;
    int32_t max_blocks, num_pages;
};

// Prefix-sharing mode. Groups are runs of consecutive sequences
// [group_start[k], group_start[k+1]) whose first shared_pages[k] block-table
// entries are the same; the group's first member's entries are used. Every
// workgroup of the fused split kernel derives both page streams from these;
// workgroup 0 stores the sums below for the merge.
struct PrefixParams {
    const int32_t *group_start;   // [num_groups + 1]
    const int32_t *shared_pages;  // [num_groups]
    int32_t *cum_own;             // [B + 1] prefix sum of steps over own (unshared) pages
    int32_t *cum_shared;          // [max_sub + 1] prefix sum of steps over shared pages per sub-group
    int32_t *seq_shared;          // [B][4] per sequence: first shared step of its sub-group in the shared
                                  // stream, shared pages, sub-group's first member, shared steps (zeros if
                                  // unshared)
    int32_t num_groups;
    int32_t max_sub;              // prefix_max_sub: bound on the sub-groups (shared-stream "sequences")
};

// Members of one shared unit: as many samples as fit kPrefixRows query rows,
// at most 16 (the tile metadata keeps members - 1 in four bits).
__host__ __device__ inline int prefix_max_members(int group) { return 16 < kPrefixRows / group ? 16 : kPrefixRows / group; }
// Bound on the sub-groups of a call: shared groups are disjoint ranges of the
// batch and a group of m members is cut into ceil(m / M) sub-groups, so there
// are at most num_groups + batch / M of them, and never more than batch.
__host__ __device__ inline int prefix_max_sub(int batch, int num_groups, int group)
{
    if (num_groups <= 0)
        return 0;
    const int bound = num_groups + batch / prefix_max_members(group);
    return bound < batch ? bound : batch;
}

struct PrefixMergeParams {
    const int32_t *seq_lens;
    const int32_t *group_start;
    const int32_t *shared_pages;
    const int32_t *cum_own;
    const int32_t *cum_shared;
    const int32_t *seq_shared;   // [B][4], as written by the split kernel
    const float *own_ml, *own_acc;        // [2 NW][G][2], [2 NW][G][D]
    const float *shared_ml, *shared_acc;  // [2 NW][kPrefixRows][2], [2 NW][kPrefixRows][D]
    const float *own_unit_ml, *own_unit_acc;        // [B Hkv][G][2 | D]: whole own units
    const float *shared_unit_ml, *shared_unit_acc;  // [B Hkv][kPrefixRows][2 | D]: whole shared units
    uint16_t *out;
    int32_t batch, max_sub, num_q_heads, num_kv_heads, group, num_workers, max_blocks;
    int32_t num_shared_workers;   // base and largest count of shared-page workgroups
    int32_t max_shared_workers;   // (effective_shared_workers)
    int32_t step_tiles;           // as the split kernel's
    int32_t fp8;
    uint32_t group_inverse;       // ceil(2^32 / group), for heads below 2^28 (unused for a group of 1)
};

struct AppendParams {
    const uint16_t *k_new;      // [B][Hkv][D] bf16 rows of the step's new token
    const uint16_t *v_new;
    const int32_t *block_table;
    const int32_t *seq_lens;    // already counting the new token
    void *k_pages;              // bf16 or E4M3 pool [num_pages][Hkv][16][D]
    void *v_pages;
    float *k_scales;            // E4M3 only: [num_pages][Hkv]
    float *v_scales;
    int32_t batch, num_kv_heads, max_blocks, num_pages;
    // Decode-engine mode (null otherwise): the step's lengths and the page of
    // every sequence's new token are read from a staging buffer laid out as
    // [lengths: B][token pages: B][block-table updates: n_upd x (slot, block,
    // page)], and the same launch also stores the lengths in set_seq_lens and
    // applies the updates to set_block_table for the attention that follows
    // (seq_lens and block_table are not read).
    const int32_t *stage;
    int32_t n_upd;
    int32_t *set_seq_lens;
    int32_t *set_block_table;
};

struct MergeParams {
    const int32_t *seq_lens;
    const int32_t *cum_pages;
    const float *part_ml;
    const float *part_acc;
    uint16_t *out;
    int32_t batch, num_q_heads, num_kv_heads, group, num_workers;
    int32_t step_tiles;   // as the split kernel's
    int32_t fp8;
    uint32_t group_inverse;   // as PrefixMergeParams'
    // Decode engine: the next step's staged append (and its bookkeeping) runs
    // in the same launch, in workgroups after the merge's, if has_next is set.
    // The merge never reads what it writes: it reads the
    // lengths only for sequences without pages, whose rows are zero whatever
    // the step (the engine's lengths are never negative).
    AppendParams next;
    int32_t has_next;
};


constexpr int kMaxPrefixBatch = 4096;      // the fused prefix kernel keeps three ints per sequence in LDS

struct PrefixWorkspace {
    int32_t *cum_own, *seq_shared, *cum_shared;
    float *own_ml, *own_acc, *shared_ml, *shared_acc;
    float *own_unit_ml, *own_unit_acc, *shared_unit_ml, *shared_unit_acc;
};
size_t prefix_workspace_layout(void *base, int batch, int max_blocks, int num_kv_heads, int group, int head_dim,
                               int num_workers, int num_groups, PrefixWorkspace *ws);

// Layout of the workspace for the given sizes; `base` may be null to size it.
size_t workspace_layout(void *base, int batch, int max_blocks, int num_kv_heads, int group,
                        int head_dim, int num_workers, Workspace *ws);

// The split kernel's dynamic LDS: the prefix sum of steps (B + 1 ints) and the
// lengths (B ints).
inline size_t split_dynamic_lds(int batch) { return sizeof(int32_t) * (2 * (size_t)batch + 1); }
// The fused prefix kernel's: for the sequences the prefix sum of own steps, the
// shared pages and the lengths (3 B + 2 ints), for the sub-groups the prefix
// sum of shared steps and the packed first member and size (2 S + 1 ints).
inline size_t prefix_dynamic_lds(int batch, int max_sub)
{
    return sizeof(int32_t) * (3 * (size_t)batch + 2 * (size_t)max_sub + 3);
}
hipError_t launch_split(const SplitParams &p, int head_dim, bool fp8, hipStream_t stream);
// Prefix mode: the own-page pass (single-unit workers) and the shared-page
// pass (one workgroup of kPrefixBlocks wavefronts per worker, one 16-row
// column block each, partial states only) in one launch, followed by the
// merge. shared.num_workers is the base count of shared workgroups and
// max_shared the largest (effective_shared_workers).
hipError_t launch_prefix_split(const SplitParams &own, const SplitParams &shared, int max_shared,
                               const PrefixParams &pp, int head_dim, bool fp8, hipStream_t stream);
hipError_t launch_merge_prefix(const PrefixMergeParams &p, int head_dim, hipStream_t stream);
hipError_t launch_merge(const MergeParams &p, int head_dim, hipStream_t stream);
hipError_t launch_append(const AppendParams &p, int head_dim, bool fp8, hipStream_t stream);
// Decode engine helper (engine.hip): fill prompt pages with synthetic data.
hipError_t launch_engine_fill(const int32_t *pages, int n_pages, int hkv, int head_dim, bool fp8, uint32_t seed,
                              void *k_pages, void *v_pages, float *k_scales, float *v_scales, hipStream_t stream);
// Pages per pipeline step of the split kernels (their streams are counted in steps).
int split_step_tiles(int head_dim, bool fp8);
// Resident split-kernel workgroups per CU (occupancy query), for the default worker count.
hipError_t split_blocks_per_cu(int head_dim, bool fp8, int *blocks);

}  // namespace sl
