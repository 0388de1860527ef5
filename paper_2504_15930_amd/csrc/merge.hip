// Log-sum-exp merge of split-KV partial states.
//
// A unit (sequence b, KV head g) whose tiles were cut across workers
// w_first..w_last left, per worker, a partial state (m_i, l_i, acc_i) for each
// of its G query heads: m_i the largest score (base-2 units), l_i the sum of
// 2^(s - m_i) and acc_i the matching un-normalised sum of value rows. With
// M = max_i m_i the exact softmax result is
//     out = sum_i 2^(m_i - M) acc_i / sum_i 2^(m_i - M) l_i
// in fp32, rounded to bf16.
//
// One wavefront per (sequence, query head). Lane i first fetches (m_i, l_i) of
// piece i, so the maximum, the weights c_i = 2^(m_i - M) and their weighted
// sum come out of two wave reductions instead of a serial walk. The rows are
// read as four columns per lane, D/4 lanes per row and so 256/D rows per load
// instruction, several loads in flight (combine_pieces): bound by the latency
// of its few dependent loads, and with long units, cut across dozens of
// workers, by how many of their rows are in flight. Units finished by a single
// worker were already written and are skipped. Sequences without pages get
// zero rows (NaN rows for an invalid negative length), which no split-KV
// worker visits.
//
// Measured (MI355X): five sequences of 2K..16K tokens, units of up to 68
// pieces: 5.3 us (one row per iteration: 18.0).
#include "append_unit.h"

namespace sl {
namespace {

typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));

typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));

// Combine the np >= 1 pieces of one row: ml_of(i) and acc_of(i) give the
// addresses of piece i's (m, l) pair and of its D accumulators. Every lane
// gets four columns, c4 = 4 (lane % (D/4)), of the un-normalised result and
// the sum of weights `l`.
template <int D, class Ml, class Acc>
__device__ __forceinline__ f32x4_t combine_pieces(int np, const Ml &ml_of, const Acc &acc_of, int lane, float &l)
{
    constexpr int kRowLanes = D / 4, kRows = kWave / kRowLanes;   // rows per load instruction
    constexpr int kFirst = 4, kMore = 8;                          // loads in flight: with the weights, and after them
    const int sub = lane / kRowLanes, c4 = 4 * (lane % kRowLanes);
    auto row = [&](int i) { return *reinterpret_cast<const f32x4_t *>(acc_of(min(i, np - 1)) + c4); };
    // The weights of up to 64 pieces and the first rows, all loads issued together.
    const f32x2_t ml0 = *reinterpret_cast<const f32x2_t *>(ml_of(min(lane, np - 1)));
    f32x4_t first[kFirst];
#pragma unroll
    for (int k = 0; k < kFirst; ++k)   // (k > 0: most units are cut in two or three)
        first[k] = k == 0 || np > kRows * k ? row(kRows * k + sub) : f32x4_t{0.f, 0.f, 0.f, 0.f};
    float M = wave_max(lane < np ? ml0[0] : -__builtin_inff());
    for (int c0 = kWave; c0 < np; c0 += kWave)   // units spread over more than 64 workers
        M = fmaxf(M, wave_max(ml_of(min(c0 + lane, np - 1))[0]));
    // Weights c_i = 2^(m_i - M); a zero weight (underflow, nothing but minus
    // infinities) drops its row.
    float c = lane < np ? __builtin_amdgcn_exp2f(ml0[0] - M) : 0.0f;
    l = wave_sum(c * ml0[1]);
    f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
    auto add = [&](float w, f32x4_t x) {
        if (w != 0.0f)
            acc += w * x;
    };
#pragma unroll
    for (int k = 0; k < kFirst; ++k)
        add(__shfl(c, kRows * k + sub, kWave), first[k]);
    for (int c0 = 0; c0 < np; c0 += kWave) {
        if (c0 > 0) {
            const f32x2_t ml = *reinterpret_cast<const f32x2_t *>(ml_of(min(c0 + lane, np - 1)));
            c = c0 + lane < np ? __builtin_amdgcn_exp2f(ml[0] - M) : 0.0f;
            l += wave_sum(c * ml[1]);
        }
        const int cnt = min(kWave, np - c0);
        for (int i = c0 == 0 ? kRows * kFirst : 0; i < cnt; i += kRows * kMore) {
            f32x4_t x[kMore];
#pragma unroll
            for (int k = 0; k < kMore; ++k)
                x[k] = row(c0 + i + kRows * k + sub);
#pragma unroll
            for (int k = 0; k < kMore; ++k) {
                const int at = i + kRows * k + sub;
                add(at < kWave ? __shfl(c, at & (kWave - 1), kWave) : 0.0f, x[k]);
            }
        }
    }
    // The rows of one instruction lie in different lanes: add them up.
#pragma unroll
    for (int off = kRowLanes; off < kWave; off <<= 1)
#pragma unroll
        for (int e = 0; e < 4; ++e)
            acc[e] += __shfl_xor(acc[e], off, kWave);
    return acc;
}

__device__ __forceinline__ uint32_t pack2(float a, float b)
{
    const f32x2_t v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}

// floor(x / y) per lane, for whole 0 <= x < 2^52 and 0 < y < 2^31 and a
// quotient below 2^31. The reciprocal is good to some 2^-52 after two Newton
// steps, so the product's floor is off by one at most, which the remainder
// (exact: every term is below 2^53) shows.
__device__ __forceinline__ int floor_div(double x, double y)
{
    double r = __builtin_amdgcn_rcp(y);
    r = __builtin_fma(r, __builtin_fma(-y, r, 1.0), r);
    r = __builtin_fma(r, __builtin_fma(-y, r, 1.0), r);
    const int q = (int)(x * r);
    const double rem = __builtin_fma(-(double)q, y, x);
    return rem < 0.0 ? q - 1 : rem >= y ? q + 1 : q;
}

// Where a unit's steps [a, a + n) (n >= 1) lie in a stream of `total` steps
// over nw workers: its first worker, how many it was cut over, and whether it
// began after the first one's first step (worker w's is floor(w total / nw),
// and floor(z) < a is z < a).
struct Cut {
    int first, pieces, odd;
};
// Of two streams at once, one division for all four ends: the lanes of a
// wavefront divide side by side. (A double quotient with its conversions is
// some hundred instructions, and with 28 wavefronts on a CU that all work one
// out, instructions set the time: with three or six of them per row the rows'
// first loads came back 2.4 (plain) and 4.4 us (prefix) into the kernel in the
// middle, 0.7 when alone.)
struct Cuts {
    Cut s, o;
};
__device__ __forceinline__ Cuts cuts_of(long long a_s, int n_s, long long tot_s, int nw_s, long long a_o, int n_o,
                                        long long tot_o, int nw_o, int lane)
{
    // Worker holding step x: the largest w with floor(w total / nw) <= x, which
    // is floor(((x + 1) nw - 1) / total).
    const bool own = (lane & 2) != 0;
    const long long end = (own ? a_o : a_s) + ((lane & 1) != 0 ? (own ? n_o : n_s) : 1);
    const double nw = own ? nw_o : nw_s, tot = __builtin_fmax((double)(own ? tot_o : tot_s), 1.0);
    const int w = floor_div(__builtin_fma((double)end, nw, -1.0), tot);
    Cuts c;
    c.s.first = __builtin_amdgcn_readlane(w, 0);
    c.s.pieces = __builtin_amdgcn_readlane(w, 1) - c.s.first + 1;
    c.s.odd = c.s.first * tot_s < a_s * nw_s ? 1 : 0;
    c.o.first = __builtin_amdgcn_readlane(w, 2);
    c.o.pieces = __builtin_amdgcn_readlane(w, 3) - c.o.first + 1;
    c.o.odd = c.o.first * tot_o < a_o * nw_o ? 1 : 0;
    return c;
}

// Head h's KV head, h / group (group_inverse: the host's ceil(2^32 / group)).
__device__ __forceinline__ int kv_head(int h, int group, uint32_t group_inverse)
{
    return group == 1 ? h : (int)(((uint64_t)(uint32_t)h * group_inverse) >> 32);
}

// NEXT: the decode engine's next-step append in the same launch (an
// AppendKind), in the workgroups after the merge's.
template <int D, int NEXT>
__global__ __launch_bounds__(kMergeThreads) void merge_kernel(MergeParams p)
{
    const int b = blockIdx.y;   // rows of workgroups: one per sequence, then the append's
    if constexpr (NEXT != kNoAppend) {
        if (b >= p.batch) {
            const int ab = (b - p.batch) * (int)gridDim.x + (int)blockIdx.x;
            apply_stage<kMergeThreads>(p.next, ab, ((int)gridDim.y - p.batch) * (int)gridDim.x);
            append_block<D, NEXT>(p.next, ab);
            return;
        }
    }
    const int Hkv = p.num_kv_heads;
    const int G = p.group;
    const int h = blockIdx.x * (kMergeThreads / kWave) + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    if (h >= p.num_q_heads)
        return;
    const int g = kv_head(h, G, p.group_inverse);
    const int j = h - g * G;
    const int lane = threadIdx.x & (kWave - 1);
    const int c4 = 4 * (lane % (D / 4));   // the lane's columns
    uint16_t *dst = p.out + ((size_t)b * p.num_q_heads + h) * D + c4;
    // First round trip: the unit's place in the stream.
    const int cb = p.cum_pages[b];
    const int nb = p.cum_pages[b + 1] - cb;
    const int len = p.seq_lens[b];
    const long long total = (long long)p.cum_pages[p.batch] * Hkv;

    if (nb == 0) {
        const uint32_t fill = len < 0 ? 0x7fc07fc0u : 0u;   // bf16 NaN / +0
        if (lane < D / 4)
            *reinterpret_cast<u32x2_t *>(dst) = u32x2_t{fill, fill};
        return;
    }
    const int NW = effective_workers(total, p.num_workers, p.step_tiles, wide_from(p.num_workers, p.fp8 != 0));
    const long long a = (long long)Hkv * cb + (long long)g * nb;   // first step of the unit
    const Cut cut = cuts_of(a, nb, total, NW, a, nb, total, NW, lane).s;
    if (cut.pieces == 1)
        return;
    // Piece i comes from worker first + i (no worker's range is empty: NW <=
    // total). Its slot is 2w, except for the unit's first worker when the unit
    // began after that worker's first step (then it was the worker's trailing
    // piece, slot 2w + 1).
    auto row_of = [&](int i) { return (size_t)(2 * (cut.first + i) + (i == 0 ? cut.odd : 0)) * G + j; };
    float l;
    const f32x4_t acc = combine_pieces<D>(
        cut.pieces, [&](int i) { return p.part_ml + 2 * row_of(i); },
        [&](int i) { return p.part_acc + row_of(i) * D; }, lane, l);
    const float inv = 1.0f / l;
    if (lane < D / 4)
        *reinterpret_cast<u32x2_t *>(dst) =
            u32x2_t{pack2(acc[0] * inv, acc[1] * inv), pack2(acc[2] * inv, acc[3] * inv)};
}

// Prefix-sharing mode: every (sequence, head) row with shared pages, or whose
// own pages were cut across workers, combines the pieces of its sub-group's
// shared unit (row member * G + head of the shared partial states) with the
// pieces of its own unit. A unit cut across workers left one piece per worker
// in the worker slots; a unit that one worker saw whole left its state in the
// unit area, at (first query row) / G. Rows finished by one worker with no
// shared pages were written by the split kernel. A sequence shorter than its
// group's shared prefix, or with an invalid length, gets a NaN row.
template <int D>
__global__ __launch_bounds__(kMergeThreads) void merge_prefix_kernel(PrefixMergeParams p)
{
    const int Hkv = p.num_kv_heads, G = p.group, Hq = p.num_q_heads;
    const int b = blockIdx.y;
    const int h = blockIdx.x * (kMergeThreads / kWave) + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    if (h >= Hq)
        return;
    const int g = kv_head(h, G, p.group_inverse);
    const int hl = h - g * G;
    const int lane = threadIdx.x & (kWave - 1);
    const int c4 = 4 * (lane % (D / 4));   // the lane's columns
    uint16_t *dst = p.out + ((size_t)b * Hq + h) * D + c4;
    // First round trip: the sequence's place in both tile streams.
    const int32_t *info = p.seq_shared + 4 * (size_t)b;   // first shared step, shared pages, lead, shared steps
    const int s_start = info[0], sk = info[1], lead = info[2], ss = info[3];
    const int L = p.seq_lens[b];
    const int co = p.cum_own[b];
    const int ob = p.cum_own[b + 1] - co;
    const long long tot_o = (long long)p.cum_own[p.batch] * Hkv;
    const long long tot_s = (long long)p.cum_shared[p.max_sub] * Hkv;
    const bool bad = L < 0 || L > p.max_blocks * kPageSize || L < sk * kPageSize;
    if (sk == 0 && ob == 0) {
        const uint32_t fill = L < 0 ? 0x7fc07fc0u : 0u;   // bf16 NaN / +0
        if (lane < D / 4)
            *reinterpret_cast<u32x2_t *>(dst) = u32x2_t{fill, fill};
        return;
    }
    const int nw_o = effective_workers(tot_o, p.num_workers, p.step_tiles, wide_from(p.num_workers, p.fp8 != 0));
    const int nw_s = effective_workers(tot_s,
                                       effective_shared_workers(tot_o, p.num_workers, p.num_shared_workers,
                                                                p.max_shared_workers, p.step_tiles, p.fp8 != 0),
                                       p.step_tiles, 0);
    const long long a_o = (long long)Hkv * co + (long long)g * ob;
    const long long a_s = (long long)Hkv * s_start + (long long)g * ss;
    const Cuts cuts = cuts_of(a_s, ss, tot_s, nw_s, a_o, ob, tot_o, nw_o, lane);   // (an empty unit's is not used)
    const int wf_o = cuts.o.first, odd_o = cuts.o.odd, n_o = ob > 0 ? cuts.o.pieces : 0;
    const int wf_s = cuts.s.first, odd_s = cuts.s.odd, n_s = sk > 0 ? cuts.s.pieces : 0;
    if (sk == 0 && n_o == 1)
        return;   // finished by a single worker
    const int row = (b - lead) * G + hl;
    const int np = n_s + n_o;
    // Pieces 0 .. n_s - 1 are the shared unit's, the others the own unit's. A
    // unit in one piece keeps its state in the unit area (an own unit of an
    // unshared sequence was written out instead: sk > 0 here). Otherwise piece
    // i of a unit is worker first + i's, in slot 2w, or 2w + 1 for its first
    // worker if the unit began after that worker's first step (no worker's
    // range is empty).
    const float *const ml_s = n_s == 1 ? p.shared_unit_ml : p.shared_ml;
    const float *const acc_s = n_s == 1 ? p.shared_unit_acc : p.shared_acc;
    const float *const ml_o = n_o == 1 ? p.own_unit_ml : p.own_ml;
    const float *const acc_o = n_o == 1 ? p.own_unit_acc : p.own_acc;
    auto row_s = [&](int i) {
        const size_t slot = n_s == 1 ? (size_t)(lead * Hkv + g) : (size_t)(2 * (wf_s + i) + (i == 0 ? odd_s : 0));
        return slot * kPrefixRows + row;
    };
    auto row_o = [&](int i) {
        const size_t slot = n_o == 1 ? (size_t)(b * Hkv + g) : (size_t)(2 * (wf_o + i) + (i == 0 ? odd_o : 0));
        return slot * G + hl;
    };
    float l;
    const f32x4_t acc = combine_pieces<D>(
        np, [&](int i) { return i < n_s ? ml_s + 2 * row_s(i) : ml_o + 2 * row_o(i - n_s); },
        [&](int i) { return i < n_s ? acc_s + row_s(i) * D : acc_o + row_o(i - n_s) * D; }, lane, l);
    const float inv = bad ? __builtin_nanf("") : 1.0f / l;
    if (lane < D / 4)
        *reinterpret_cast<u32x2_t *>(dst) =
            u32x2_t{pack2(acc[0] * inv, acc[1] * inv), pack2(acc[2] * inv, acc[3] * inv)};
}

}  // namespace

hipError_t launch_merge(const MergeParams &p, int head_dim, hipStream_t stream)
{
    const int per_block = kMergeThreads / kWave;
    static_assert(kMergeThreads == kAppendThreads, "the append's workgroups ride in the merge's launch");
    const AppendKind kind = p.has_next ? append_kind(p.next, p.fp8 != 0) : kNoAppend;
    const long long next_blocks = p.has_next ? append_blocks(p.next, kind) : 0;
    // A grid has at most 65535 rows; with few heads and thousands of sequences
    // the append's workgroups take wider ones (the merge's beyond the heads exit).
    unsigned x = (unsigned)((p.num_q_heads + per_block - 1) / per_block);
    while (p.batch + (next_blocks + x - 1) / x > 65535)
        x *= 2;
    const dim3 grid(x, (unsigned)(p.batch + (next_blocks + x - 1) / x));
    const dim3 block(kMergeThreads);
#define SL_MERGE(DD, NN) \
    if (head_dim == DD && kind == NN) \
        hipLaunchKernelGGL((merge_kernel<DD, NN>), grid, block, 0, stream, p); \
    else
    SL_MERGE(128, kNoAppend)
    SL_MERGE(128, kAppendBf16)
    SL_MERGE(128, kAppendSpread)
    SL_MERGE(128, kAppendWave)
    SL_MERGE(64, kNoAppend)
    SL_MERGE(64, kAppendBf16)
    SL_MERGE(64, kAppendSpread)
    SL_MERGE(64, kAppendWave)
        return hipErrorInvalidValue;
#undef SL_MERGE
    return hipGetLastError();
}

hipError_t launch_merge_prefix(const PrefixMergeParams &p, int head_dim, hipStream_t stream)
{
    const int per_block = kMergeThreads / kWave;
    const dim3 grid((unsigned)((p.num_q_heads + per_block - 1) / per_block), (unsigned)p.batch);
    if (head_dim == 128)
        hipLaunchKernelGGL(merge_prefix_kernel<128>, grid, dim3(kMergeThreads), 0, stream, p);
    else if (head_dim == 64)
        hipLaunchKernelGGL(merge_prefix_kernel<64>, grid, dim3(kMergeThreads), 0, stream, p);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace sl
