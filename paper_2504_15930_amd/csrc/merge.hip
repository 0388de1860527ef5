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
// One wavefront per (unit, query head). Lane i first fetches (m_i, l_i) of
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
    for (int k = 0; k < kFirst; ++k)
        first[k] = row(kRows * k + sub);
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

// floor(x / y) for 0 <= x < 2^53, 0 < y < 2^31: a double quotient corrected by
// one step (64-bit integer division is a long software sequence on the GPU).
__device__ __forceinline__ long long div_floor(long long x, long long y)
{
    long long q = (long long)((double)x / (double)y);
    if (q * y > x)
        --q;
    else if ((q + 1) * y <= x)
        ++q;
    return q;
}

// NEXT: the decode engine's next-step append in the same launch (0 none,
// 1 bf16 cache, 2 E4M3 cache), in the workgroups after the merge's.
template <int D, int NEXT>
__global__ __launch_bounds__(kMergeThreads) void merge_kernel(MergeParams p, int merge_blocks)
{
    if constexpr (NEXT != 0) {
        if ((int)blockIdx.x >= merge_blocks) {
            const int ab = (int)blockIdx.x - merge_blocks;
            apply_stage(p.next, ab * kMergeThreads + threadIdx.x, ((int)gridDim.x - merge_blocks) * kMergeThreads);
            append_block<D, NEXT == 2>(p.next, ab);
            return;
        }
    }
    const int Hkv = p.num_kv_heads;
    const int G = p.group;
    const int item = blockIdx.x * (kMergeThreads / kWave) +
                     __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    if (item >= p.batch * Hkv * G)
        return;
    const int u = item / G;
    const int j = item - u * G;
    const int b = u / Hkv;
    const int g = u - b * Hkv;
    const int lane = threadIdx.x & (kWave - 1);
    const int c4 = 4 * (lane % (D / 4));   // the lane's columns
    uint16_t *dst = p.out + ((size_t)b * p.num_q_heads + (size_t)g * G + j) * D + c4;
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
    const long long NW = effective_workers(total, p.num_workers, p.step_tiles);
    const long long a = (long long)Hkv * cb + (long long)g * nb;   // first step of the unit
    const long long e = a + nb;                                    // one past its last step
    // Worker holding step x: the largest w with floor(w * total / NW) <= x.
    const int wf = (int)div_floor((a + 1) * NW - 1, total);
    const int wl = (int)div_floor(e * NW - 1, total);
    if (wf == wl)
        return;
    const int np = wl - wf + 1;
    // Piece i comes from worker wf + i (no worker's range is empty: NW <=
    // total). Its slot is 2w, except for the unit's first worker when the unit
    // began after that worker's first step (then it was the worker's trailing
    // piece, slot 2w + 1).
    const int odd = div_floor((long long)wf * total, NW) < a ? 1 : 0;
    auto row_of = [&](int i) { return (size_t)(2 * (wf + i) + (i == 0 ? odd : 0)) * G + j; };
    float l;
    const f32x4_t acc = combine_pieces<D>(
        np, [&](int i) { return p.part_ml + 2 * row_of(i); }, [&](int i) { return p.part_acc + row_of(i) * D; }, lane, l);
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
    const int item = blockIdx.x * (kMergeThreads / kWave) + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    if (item >= p.batch * Hq)
        return;
    const int b = item / Hq;
    const int h = item - b * Hq;
    const int g = h / G;
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
    const long long nw_o = effective_workers(tot_o, p.num_workers, p.step_tiles);
    const long long a_o = (long long)Hkv * co + (long long)g * ob;
    int wf_o = 0, n_o = 0;
    if (ob > 0) {
        wf_o = (int)div_floor((a_o + 1) * nw_o - 1, tot_o);
        n_o = (int)div_floor((a_o + ob) * nw_o - 1, tot_o) - wf_o + 1;
    }
    if (sk == 0 && n_o == 1)
        return;   // finished by a single worker
    const long long nw_s =
        tot_s > 0 ? effective_workers(tot_s,
                                      effective_shared_workers(tot_o, p.num_workers, p.num_shared_workers,
                                                               p.max_shared_workers, p.step_tiles),
                                      p.step_tiles)
                  : 1;
    long long a_s = 0;
    int wf_s = 0, n_s = 0, row = 0;
    if (sk > 0) {
        a_s = (long long)Hkv * s_start + (long long)g * ss;
        wf_s = (int)div_floor((a_s + 1) * nw_s - 1, tot_s);
        n_s = (int)div_floor((a_s + ss) * nw_s - 1, tot_s) - wf_s + 1;
        row = (b - lead) * G + hl;
    }
    const int np = n_s + n_o;
    // Pieces 0 .. n_s - 1 are the shared unit's, the others the own unit's. A
    // unit in one piece keeps its state in the unit area (an own unit of an
    // unshared sequence was written out instead: sk > 0 here). Otherwise piece
    // i of a unit is worker wf + i's, in slot 2w, or 2w + 1 for its first worker
    // if the unit began after that worker's first step (no worker's range is
    // empty).
    const int odd_s = sk > 0 && div_floor(wf_s * tot_s, nw_s) < a_s ? 1 : 0;
    const int odd_o = ob > 0 && div_floor(wf_o * tot_o, nw_o) < a_o ? 1 : 0;
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
    const long long items = (long long)p.batch * p.num_kv_heads * p.group;
    const int per_block = kMergeThreads / kWave;
    const int merge_blocks = (int)((items + per_block - 1) / per_block);
    static_assert(kMergeThreads == kAppendThreads, "the append's workgroups ride in the merge's launch");
    int next_blocks = 0;
    if (p.next_kind != 0) {
        const long long units = (long long)p.next.batch * p.next.num_kv_heads;
        next_blocks = (int)(p.next_kind == 2 ? append_blocks<true>(units) : append_blocks<false>(units));
    }
    const dim3 grid((unsigned)(merge_blocks + next_blocks));
    const dim3 block(kMergeThreads);
#define SL_MERGE(DD, NN) hipLaunchKernelGGL((merge_kernel<DD, NN>), grid, block, 0, stream, p, merge_blocks)
    if (head_dim == 128 && p.next_kind == 0)
        SL_MERGE(128, 0);
    else if (head_dim == 128 && p.next_kind == 1)
        SL_MERGE(128, 1);
    else if (head_dim == 128 && p.next_kind == 2)
        SL_MERGE(128, 2);
    else if (head_dim == 64 && p.next_kind == 0)
        SL_MERGE(64, 0);
    else if (head_dim == 64 && p.next_kind == 1)
        SL_MERGE(64, 1);
    else if (head_dim == 64 && p.next_kind == 2)
        SL_MERGE(64, 2);
    else
        return hipErrorInvalidValue;
#undef SL_MERGE
    return hipGetLastError();
}

}  // namespace sl

namespace sl {

hipError_t launch_merge_prefix(const PrefixMergeParams &p, int head_dim, hipStream_t stream)
{
    const long long items = (long long)p.batch * p.num_q_heads;
    const int per_block = kMergeThreads / kWave;
    const dim3 grid((unsigned)((items + per_block - 1) / per_block));
    if (head_dim == 128)
        hipLaunchKernelGGL(merge_prefix_kernel<128>, grid, dim3(kMergeThreads), 0, stream, p);
    else if (head_dim == 64)
        hipLaunchKernelGGL(merge_prefix_kernel<64>, grid, dim3(kMergeThreads), 0, stream, p);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace sl
