#ifndef SL_APPEND_UNIT_H
#define SL_APPEND_UNIT_H
// KV append for one decode step: every sequence's new key/value rows join its
// paged cache before the step's attention reads it.
//
// With L = seq_lens[b] already counting the new token, the token t = L - 1
// goes to page block_table[b][t / 16], slot t % 16, for every KV head.
//
// bf16 cache: the row is stored as is.
//
// E4M3 cache (one fp32 scale per (page, KV head) for K and one for V; the
// cached value is decode(code) * scale): the scale of a page-head tile only
// grows. With a = max |x| over the row (NaN elements ignored):
//   slot 0 (fresh page)          s = a / 448 (1 if a == 0)
//   a <= s_old * 448             s = s_old
//   a >  s_old * 448             s = a / 448 and every earlier slot j of the
//                                tile is re-encoded: c = enc(decode(c) * s_old / s)
// and the new row is enc(x / s). enc() rounds to nearest even and saturates
// to +-448 (NaN -> 0x7F). All of it is binary32 arithmetic in that order, so
// the codes are reproducible bit for bit.
//
// bf16: one wavefront per (sequence, KV head). E4M3: four wavefronts for its K
// tile and four for its V tile, each re-encoding four of the tile's rows, or
// with many units one wavefront for both tiles (kSpreadUnits). Lane l holds
// elements [l * D/64, (l + 1) * D/64) of the new row. The data per call is a
// few KB per unit, so with few units the kernel is bound by the latency of its
// dependent loads (length -> block table -> scale and codes) and by the
// arithmetic of a re-encoded tile (2048 true divisions and saturating
// conversions): for 96 sequences x 4 heads (MI355X) one wavefront per unit that
// did K, then V took 6.4 us, eight wavefronts that fetch the old codes with the
// scale 3.9.
#include <type_traits>

#include "sl_internal.h"
#include "wave_ops.h"

namespace sl {
namespace {


typedef short i16x2_t __attribute__((ext_vector_type(2)));

// One E4M3 code -> binary32, exact (the bf16 conversion covers every code).
__device__ __forceinline__ float e4m3_to_f32(uint32_t code)
{
    const uint32_t w = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(code, 1.0f, false));
    return __builtin_bit_cast(float, w << 16);
}

// Signed-zero code of y if y rounds to zero in E4M3 (|y| <= 2^-10, half the
// smallest subnormal, a tie that goes to the even code 0), else 0xffffffff.
__device__ __forceinline__ uint32_t e4m3_zero_code(float y)
{
    const uint32_t u = __builtin_bit_cast(uint32_t, y);
    return (u & 0x7fffffffu) <= 0x3a800000u ? (u >> 24) & 0x80u : 0xffffffffu;
}

// Two binary32 values -> two E4M3 codes (low byte: a). Clamped to +-448
// first, so the conversion never overflows; NaN maps to 0x7F. Magnitudes up
// to 2^-10 (fp32 denormals among them, which the conversion does not round
// like other inputs) are encoded as signed zero directly.
__device__ __forceinline__ uint32_t f32x2_to_e4m3(float a, float b)
{
    const float ca = __builtin_fminf(__builtin_fmaxf(a, -448.0f), 448.0f);
    const float cb = __builtin_fminf(__builtin_fmaxf(b, -448.0f), 448.0f);
    const i16x2_t r = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(i16x2_t{0, 0}, ca, cb, 1.0f, false);
    uint32_t lo = (uint32_t)(uint16_t)r[0];
    const uint32_t za = e4m3_zero_code(a), zb = e4m3_zero_code(b);
    if (za != 0xffffffffu)
        lo = (lo & 0xff00u) | za;
    if (zb != 0xffffffffu)
        lo = (lo & 0x00ffu) | (zb << 8);
    if (a != a)
        lo = (lo & 0xff00u) | 0x7fu;
    if (b != b)
        lo = (lo & 0x00ffu) | 0x7f00u;
    return lo;
}

// Quantise-on-write of one row into one page-head tile (16 x D codes), by P
// wavefronts (`part` 0 .. P - 1; part k owns the tile's rows 16 k / P and on)
// in two phases. load_row() and load_tile() fetch the row, the scale and, with
// several parts, the part's old codes, all in flight together; store() works
// out the new scale, the same in every part, re-encodes the part's earlier
// rows if it grew, and writes the new row in the part that owns its slot.
// Since store() overwrites the scale and the codes that load_tile() reads,
// every part's load must have returned before any part's store: landed() and
// a barrier. One wavefront alone fetches the old codes only once it knows that
// the scale grows.
template <int D, int P>
struct AppendTile {
    static constexpr int E = D / kWave;             // row elements per lane (1 or 2)
    static constexpr int kRows = kPageSize / P;     // rows per part
    // The part's old codes: a lane's own run of dwords with several parts (one
    // load), a row after the other for one wavefront alone, which skips those
    // past the slot.
    using Word = std::conditional_t<(P > 1), uint32_t, std::conditional_t<D == 128, uint16_t, uint8_t>>;
    static constexpr int kCodes = sizeof(Word);                 // codes per word
    static constexpr int W = kRows * D / (kCodes * kWave);      // words per lane
    __device__ static constexpr int word(int w, int lane) { return P > 1 ? W * lane + w : kWave * w + lane; }
    uint32_t x;
    float s_old;
    Word old[P > 1 ? W : 1];

    __device__ __forceinline__ void load_row(const uint16_t *row, int lane)
    {
        if constexpr (E == 2)
            x = reinterpret_cast<const uint32_t *>(row)[lane];
        else
            x = row[lane];
    }
    __device__ __forceinline__ void load_tile(const uint8_t *tile, const float *scale, int part, int lane)
    {
        s_old = *scale;
        if constexpr (P > 1) {
            const Word *codes = reinterpret_cast<const Word *>(tile + kRows * part * D);
#pragma unroll
            for (int w = 0; w < W; ++w)
                old[w] = codes[word(w, lane)];
        }
    }
    // Every load of load_tile() has returned, and its value is what store()
    // uses: for the compiler the registers change here. (A barrier alone does
    // not say so. The address of the scale is the same for the whole wavefront
    // and this wavefront has stored nothing yet, so the compiler made it a
    // scalar load and moved it to its first use, behind the barrier, where
    // another part may have stored the grown scale already.)
    __device__ __forceinline__ void landed()
    {
        asm volatile("" : "+v"(s_old));
#pragma unroll
        for (int w = 0; w < (P > 1 ? W : 0); ++w)
            asm volatile("" : "+v"(old[w]));
    }
    __device__ __forceinline__ void store(uint8_t *tile, float *scale, int slot, int part, int lane) const
    {
        float v[E];
        v[0] = __builtin_bit_cast(float, x << 16);
        if constexpr (E == 2)
            v[1] = __builtin_bit_cast(float, x & 0xffff0000u);
        // NaN elements do not count towards the maximum. A comparison skips every
        // NaN (fmax would return a quiet NaN for a signalling one and lose the
        // other operand), so only finite or infinite magnitudes reach the wave max.
        float a = 0.0f;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const float m = __builtin_fabsf(v[e]);
            a = m > a ? m : a;
        }
        a = wave_max(a);

        float s;
        if (slot == 0) {
            s = a > 0.0f ? a / 448.0f : 1.0f;
        } else if (a <= s_old * 448.0f) {
            s = s_old;
        } else {
            s = a / 448.0f;
            // Re-encode the part's earlier rows with the grown scale.
            Word *codes = reinterpret_cast<Word *>(tile + kRows * part * D);
            auto earlier = [&](int w) { return kRows * part + kCodes * word(w, lane) / D < slot; };
            uint32_t was[W];   // (set where it is read; zeros elsewhere would be waited for at the first load)
#pragma unroll
            for (int w = 0; w < W; ++w) {
                if constexpr (P > 1)
                    was[w] = old[w];
                else if (earlier(w))
                    was[w] = codes[word(w, lane)];
            }
#pragma unroll
            for (int w = 0; w < W; ++w) {
                if (!earlier(w))
                    continue;
                uint32_t now = 0;
#pragma unroll
                for (int c = 0; c < kCodes; c += 2) {
                    const float r0 = (e4m3_to_f32(was[w] >> (8 * c) & 0xffu) * s_old) / s;
                    const float r1 = kCodes > 1 ? (e4m3_to_f32(was[w] >> (8 * c + 8) & 0xffu) * s_old) / s : 0.0f;
                    now |= (f32x2_to_e4m3(r0, r1) & 0xffffu) << (8 * c);
                }
                codes[word(w, lane)] = (Word)now;
            }
        }
        if (part == slot / kRows) {
            if constexpr (E == 2)
                *reinterpret_cast<uint16_t *>(tile + slot * D + 2 * lane) =
                    (uint16_t)f32x2_to_e4m3(v[0] / s, v[1] / s);
            else
                tile[slot * D + lane] = (uint8_t)f32x2_to_e4m3(v[0] / s, 0.0f);
            if (lane == 0)
                *scale = s;
        }
    }
};

constexpr int kMaxApplyBlocks = 4096;

// The engine's bookkeeping for a step (staged mode only): store the step's
// lengths in set_seq_lens and apply its block-table updates, spread over the
// first of the launch's `blocks` workgroups (THREADS threads each), of which
// this one is `blk`: enough of them for any step, and few enough that a thread's
// index fits 32 bits. Indices were checked by the engine.
template <int THREADS>
__device__ __forceinline__ void apply_stage(const AppendParams &p, int blk, int blocks)
{
    blocks = min(blocks, kMaxApplyBlocks);
    if (blk >= blocks)
        return;
    const int nthreads = blocks * THREADS;
    const int first = blk * THREADS + (int)threadIdx.x;
    for (int i = first; i < p.batch; i += nthreads)
        p.set_seq_lens[i] = p.stage[i];
    for (int i = first; i < p.n_upd; i += nthreads) {
        const int32_t *u = p.stage + 2 * p.batch + 3 * i;
        p.set_block_table[(size_t)u[0] * p.max_blocks + u[1]] = u[2];
    }
}

// Whether token L - 1 of a sequence of length L (the new token included) is
// appended to page `page`: an invalid length or page id leaves the cache
// untouched.
__device__ __forceinline__ bool append_valid(const AppendParams &p, int L, int page)
{
    return L > 0 && L <= p.max_blocks * kPageSize && page >= 0 && page < p.num_pages;
}

// One of the K (`which` 0) and V (1) rows of unit `unit` = b * Hkv + g into
// an E4M3 cache, by P wavefronts (part 0 .. P - 1): AppendTile's two phases.
template <int D, int P>
struct AppendE4m3 {
    AppendTile<D, P> t;
    uint8_t *tile;
    float *scale;

    __device__ __forceinline__ void load_row(const AppendParams &p, int unit, int which, int lane)
    {
        t.load_row((which ? p.v_new : p.k_new) + (size_t)unit * D, lane);
    }
    __device__ __forceinline__ void load_tile(const AppendParams &p, int g, int which, int page, int part, int lane)
    {
        const size_t at = (size_t)page * p.num_kv_heads + g;   // page-head tile index
        tile = static_cast<uint8_t *>(which ? p.v_pages : p.k_pages) + at * kPageSize * D;
        scale = (which ? p.v_scales : p.k_scales) + at;
        t.load_tile(tile, scale, part, lane);
    }
    __device__ __forceinline__ void landed() { t.landed(); }
    __device__ __forceinline__ void store(int L, int part, int lane) const
    {
        t.store(tile, scale, (L - 1) % kPageSize, part, lane);
    }
};

// Length (new token included) of sequence b and the page of its new token:
// from the staging buffer, or from the lengths array and the block table (-1
// for a length that has no table entry).
__device__ __forceinline__ void append_place(const AppendParams &p, int b, int &L, int &page)
{
    if (p.stage) {   // both across the host link: fetched together
        L = p.stage[b];
        page = p.stage[p.batch + b];
        return;
    }
    L = p.seq_lens[b];
    page = L > 0 && L <= p.max_blocks * kPageSize
               ? p.block_table[(size_t)b * p.max_blocks + (L - 1) / kPageSize]
               : -1;
}

// Workgroups of kAppendThreads threads that append a step's rows. bf16 cache:
// a wavefront per unit. E4M3: up to kSpreadUnits units, a workgroup per unit
// and K or V; beyond them a wavefront per unit, which fills the chip just as
// well and fetches the old codes (4 KB per unit of D = 128) only where the
// scale grows. Spread -> one wavefront, calls of D = 128, MI355X:
//   units                2048           3072           4096           16384         65536
//   no scale grows        9.0 -> 9.1     9.5 -> 9.0    11.1 -> 9.1    36.6 -> 9.2   166 -> 25 us
//   one scale in five     8.3 -> 9.6     9.6 -> 10.8   11.8 -> 12.0          22.0          60
//   every scale          10.2 -> 10.4   13.5 -> 13.0   16.9 -> 15.2          36.9         116
// Each is a kernel of its own: together their code reached the merge's launch,
// whose append has 1024 units for 256 sequences x 4 heads, 1.3 us later.
constexpr int kAppendThreads = 256;
constexpr int kSpreadUnits = 2048;
enum AppendKind { kNoAppend, kAppendBf16, kAppendSpread, kAppendWave };
inline AppendKind append_kind(const AppendParams &p, bool fp8)
{
    return !fp8 ? kAppendBf16 : (long long)p.batch * p.num_kv_heads <= kSpreadUnits ? kAppendSpread : kAppendWave;
}
inline long long append_blocks(const AppendParams &p, AppendKind kind)
{
    const long long units = (long long)p.batch * p.num_kv_heads;
    return kind == kAppendSpread ? 2 * units : (units + kAppendThreads / kWave - 1) / (kAppendThreads / kWave);
}

// Both rows of unit `unit` into a bf16 cache, by one wavefront.
template <int D>
__device__ __forceinline__ void append_unit_bf16(const AppendParams &p, int unit, int lane)
{
    static_assert(D / 2 <= kWave, "one dword of each row per lane");
    uint32_t kw = 0, vw = 0;
    if (lane < D / 2) {   // beside the length and the page
        kw = reinterpret_cast<const uint32_t *>(p.k_new + (size_t)unit * D)[lane];
        vw = reinterpret_cast<const uint32_t *>(p.v_new + (size_t)unit * D)[lane];
    }
    const int b = unit / p.num_kv_heads;
    int L, page;
    append_place(p, b, L, page);
    if (!append_valid(p, L, page) || lane >= D / 2)
        return;
    const size_t tile = (size_t)page * p.num_kv_heads + (unit - b * p.num_kv_heads);
    const size_t row = (tile * kPageSize + (L - 1) % kPageSize) * D;
    reinterpret_cast<uint32_t *>(static_cast<uint16_t *>(p.k_pages) + row)[lane] = kw;
    reinterpret_cast<uint32_t *>(static_cast<uint16_t *>(p.v_pages) + row)[lane] = vw;
}

// Both rows of unit `unit` into an E4M3 cache, by one wavefront.
template <int D>
__device__ __forceinline__ void append_unit_e4m3(const AppendParams &p, int unit, int lane)
{
    AppendE4m3<D, 1> k, v;
    k.load_row(p, unit, 0, lane);   // beside the length and the page
    v.load_row(p, unit, 1, lane);
    const int b = unit / p.num_kv_heads;
    int L, page;
    append_place(p, b, L, page);
    if (!append_valid(p, L, page))
        return;
    k.load_tile(p, unit - b * p.num_kv_heads, 0, page, 0, lane);
    v.load_tile(p, unit - b * p.num_kv_heads, 1, page, 0, lane);
    k.store(L, 0, lane);
    v.store(L, 0, lane);
}

// Workgroup `blk` of append_blocks, run by its kAppendThreads threads.
template <int D, int KIND>
__device__ __forceinline__ void append_block(const AppendParams &p, int blk)
{
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = threadIdx.x & (kWave - 1);
    const int units = p.batch * p.num_kv_heads;
    if constexpr (KIND == kAppendSpread) {
        const int unit = blk >> 1, which = blk & 1;
        if (unit >= units)
            return;
        const int b = unit / p.num_kv_heads;
        AppendE4m3<D, 4> a;
        a.load_row(p, unit, which, lane);   // beside the length and the page
        int L, page;
        append_place(p, b, L, page);
        if (!append_valid(p, L, page))      // the same for the whole workgroup
            return;
        a.load_tile(p, unit - b * p.num_kv_heads, which, page, wave, lane);
        a.landed();
        __syncthreads();
        a.store(L, wave, lane);
    } else {
        const int unit = blk * (kAppendThreads / kWave) + wave;
        if (unit >= units)
            return;
        if constexpr (KIND == kAppendWave)
            append_unit_e4m3<D>(p, unit, lane);
        else
            append_unit_bf16<D>(p, unit, lane);
    }
}

}  // namespace
}  // namespace sl

#endif  // SL_APPEND_UNIT_H
