#ifndef SL_DECODE_UNIT_H
#define SL_DECODE_UNIT_H
// Split-KV decode attention worker for gfx950.
//
// One wavefront is one worker. It streams its contiguous range of page-head
// tiles (see sl_internal.h) as a flat sequence, keeping an online-softmax
// state for the G query heads of the unit (sequence, KV head) the current tile
// belongs to, and finishing that unit whenever its last tile, or the end of
// the range, is reached. For the shared pages of prefix-shared attention the
// four wavefronts of a workgroup stream the same range, each computing one
// 16-row column block of the shared unit's query rows (kSharedPages).
//
// Per 16-token tile, with lane = n + 16 * quad (n = lane & 15, quad = lane >> 4):
//
//   scores  S^T[t][j] = sum_d K[t][d] Q[j][d]       v_mfma_f32_16x16x32_bf16
//           A = K   (row t = n, 8 consecutive d per lane; the tile is read as
//                    whole 1 KB runs and regrouped through LDS)
//           B = Q^T (column j = n; query rows j >= G are zero padding)
//           -> lane (j, quad) holds the scores of head j for tokens 4 quad + r
//   softmax running max / sum per head j, kept in the lanes of column j: the
//           only cross-lane step is a max over the four quads of a column
//   values  O^T[d][j] += sum_t V[t][d] P[j][t]       v_mfma_f32_16x16x16bf16_1k
//           (two tiles of a step at once: v_mfma_f32_16x16x32_bf16)
//           A = V^T (lane (n, quad) holds V[4 quad + r][d_i(n)] for r = 0..3,
//                    gathered from four 16-byte row loads and repacked)
//           B = P^T exactly as the score MFMA left it (no data movement)
//           -> lane (j, quad) accumulates O[j][d] for D/4 consecutive d
//
// V goes straight from HBM into MFMA operand registers: its loads already
// cover whole 128-byte lines. The K operand layout would read only half a
// line per instruction (each row spread over four lanes), which streams at
// ~6.0 TB/s instead of ~6.85 TB/s on MI355X, so K is read in whole 1 KB runs
// and regrouped through a small per-wave LDS buffer. Both are streamed with
// non-temporal loads. A worker goes through its range in steps of one, two or
// four tiles (step_tiles), software-pipelined; the steps' units, pages and
// block-table entries are worked out 64 at a time, one per lane, ahead of the
// steps themselves, and the query rows of a unit are loaded together with the
// unit's first step, so the stream never waits on a dependent load, also
// across unit boundaries.
//
// FP8 pages hold OCP E4M3 codes; they are widened to bf16 exactly
// (v_cvt_scalef32_pk_bf16_fp8 with unit scale), the per-(page, head) key
// scale multiplies the fp32 scores and the value scale multiplies the
// probabilities before they are rounded for the value MFMA.
#include "sl_internal.h"
#include "wave_ops.h"

namespace sl {
namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef short i16x4_t __attribute__((ext_vector_type(4)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));

constexpr float kNegInf = -__builtin_inff();
// A partial state l = sum 2^(s - m), acc = sum 2^(s - m) v is exact for any
// reference m. The running maximum is raised only when a score exceeds it by
// more than this slack (base-2 units), which bounds the weights by 2^8 and
// leaves the accumulators untouched on most tiles after a unit's first.
constexpr float kRescaleSlack = 8.0f;
// Tiles per pipeline step and steps in flight. A worker is one wavefront, most
// often alone on its SIMD, so its chain of dependent instructions per tile is
// time that nothing fills: at 1024 workers a wavefront has ~0.65 us for an
// E4M3 tile of 4 KB before HBM waits for it. Two tiles per step share the
// bookkeeping, the look at the running maximum and half of the value MFMAs
// (compute_step); a step then carries as many bytes as one bf16 tile of D =
// 128, which is HBM-bound with one tile per step (two measured the same to 1%
// slower). Step (split + merge) with one tile -> this choice, MI355X:
//   bf16 D = 64, 384 x 1..2048 tokens, 8 KV heads   165 -> 130 us (with 1024 workers)
//   E4M3 D = 128, 512 x 512 + lognormal(2048)        319 -> 316 us; at 768 workers 381 -> 327
//   E4M3 D = 64, 384 x 1..4096 tokens, 8 KV heads   226 -> 146 us (two tiles: 157)
// Two steps in flight; three were no faster anywhere (and slower where they
// cost a resident workgroup, in the prefix kernel).
template <int D, bool FP8>
constexpr int step_tiles() { return D == 64 ? (FP8 ? 4 : 2) : (FP8 ? 2 : 1); }
constexpr int kPipelineDepth = 2;
constexpr int kRawBufferWord3 = 0x00020000;  // untyped 32-bit buffer resource (CDNA3/4)

// Two fp32 -> packed bf16 pair, round to nearest even (v_cvt_pk_bf16_f32).
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi)
{
    f32x2_t v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __builtin_bit_cast(float, w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __builtin_bit_cast(float, w & 0xffff0000u); }

// Four E4M3 codes (one dword) -> four bf16 (two dwords), exact.
__device__ __forceinline__ void e4m3x4_to_bf16(uint32_t codes, uint32_t &lo, uint32_t &hi)
{
    lo = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(codes, 1.0f, false));
    hi = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(codes, 1.0f, true));
}

// Max / sum over the lanes n, n + 16, n + 32, n + 48 of a column.
// (The gfx950 lane-swap builtins would avoid the LDS crossbar here, but this
// compiler folds max(h[0], h[1]) of their two results to one of them, so the
// plain shuffles are used.)
__device__ __forceinline__ float quad_max(float x)
{
    x = fmaxf(x, __shfl_xor(x, 16, kWave));
    return fmaxf(x, __shfl_xor(x, 32, kWave));
}
__device__ __forceinline__ float quad_sum(float x)
{
    x += __shfl_xor(x, 16, kWave);
    return x + __shfl_xor(x, 32, kWave);
}

template <int D, bool FP8>
struct Tile {
    // Per-lane dwords of K (score-MFMA A operands) and V (four rows).
    static constexpr int KW = FP8 ? D / 16 : D / 8;
    static constexpr int VW = FP8 ? D / 16 : D / 8;
    uint32_t k[KW];
    uint32_t v[VW];
    float scl;           // FP8: key scale in lanes 0-31, value scale in lanes 32-63
};

// One pipeline step: NT consecutive tiles of one unit (fewer at the unit's end).
template <int D, bool FP8, int NT>
struct Step {
    Tile<D, FP8> t[NT];
    u32x4_t q[D / 32];   // the unit's query rows, loaded with a unit's first step only
    uint32_t meta;       // metadata (kMeta* bits, wave-uniform)
    int32_t valid;       // live tokens of the step, 1 .. 16 NT; kSharedPages: | (members - 1) << 8
};

// Query element index held by (quad, item) in k-step s; must match k_operand.
template <int D, bool FP8>
__device__ __forceinline__ int q_index(int s, int quad)
{
    return FP8 ? quad * (D / 4) + 8 * s : 32 * s + 8 * quad;
}

// K/V pages are read exactly once per call: stream them with non-temporal loads
// so they do not displace reusable lines in L2 / the Infinity Cache (measured on
// MI355X: random 4 KB tiles reach ~6.8 TB/s this way, ~6.0 TB/s with plain loads).
constexpr int kCachePolicyStream = 2;   // NT

__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const void *base, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, (int)bytes, kRawBufferWord3);
}

// The score-MFMA B operands of a unit with first query row row0, zero where
// `with_q` is false: lane (n, quad) takes query row n, and the rows past the
// group's G lie past the resource's end, so they are zero too.
template <int D, bool FP8>
__device__ __forceinline__ void load_q(u32x4_t (&q)[D / 32], const SplitParams &p, uint32_t row0, bool with_q, int n,
                                       int quad)
{
    const __amdgpu_buffer_rsrc_t qr = buffer_of(p.q + (size_t)row0 * D, with_q ? (uint32_t)(p.group * D * 2) : 0u);
#pragma unroll
    for (int s = 0; s < D / 32; ++s)
        q[s] = __builtin_bit_cast(
            u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(qr, 2 * (n * D + q_index<D, FP8>(s, quad)), 0, 0));
}

// Issue the K/V loads of one tile (page-head tile index `tile`), always the
// same number of them: the compiler's counter waits can then tell the loads of
// one step from those of the next. (A load issued on some paths only makes
// every later wait assume the path with the fewest, and so drain loads that
// should stay in flight.) What must not be read (`read` false: a tile past the
// range, a page outside the pool) goes through a buffer resource of zero
// bytes, whose loads return zeros without touching memory.
//
// K/V are streamed with non-temporal loads (STREAM) unless the tile is read by
// several wavefronts at once (the column blocks of a shared unit), where plain
// loads let the siblings find it in L2.
template <int D, bool FP8, bool STREAM>
__device__ __forceinline__ void issue_tile(Tile<D, FP8> &t, const SplitParams &p, uint32_t tile_index, bool read,
                                           int n, int quad, int lane)
{
    constexpr int kPolicy = STREAM ? kCachePolicyStream : 0;
    constexpr uint32_t kTileBytes = kPageSize * D * (FP8 ? 1 : 2);
    const size_t tile = tile_index;
    const __amdgpu_buffer_rsrc_t kt =
        buffer_of(static_cast<const uint8_t *>(p.k_pages) + tile * kTileBytes, read ? kTileBytes : 0u);
    const __amdgpu_buffer_rsrc_t vt =
        buffer_of(static_cast<const uint8_t *>(p.v_pages) + tile * kTileBytes, read ? kTileBytes : 0u);
    // K: whole 1 KB runs per instruction (lane l reads bytes 16 l of each
    // run), so every instruction covers complete 128-byte lines; the rows are
    // regrouped into the score-MFMA layout through LDS when the tile is used.
#pragma unroll
    for (int i = 0; i < Tile<D, FP8>::KW / 4; ++i) {
        const u32x4_t x = __builtin_bit_cast(
            u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(kt, 16 * lane + 1024 * i, 0, kPolicy));
#pragma unroll
        for (int c = 0; c < 4; ++c)
            t.k[4 * i + c] = x[c];
    }
    // V: lane (n, quad) reads D/16 consecutive elements of rows 4 quad + r.
    constexpr int kRow = D * (FP8 ? 1 : 2);
    const int voff = 4 * quad * kRow + n * (kRow / 16);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        if constexpr (kRow == 256) {
            const u32x4_t x = __builtin_bit_cast(
                u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(vt, voff + r * kRow, 0, kPolicy));
#pragma unroll
            for (int c = 0; c < 4; ++c)
                t.v[4 * r + c] = x[c];
        } else if constexpr (kRow == 128) {
            const u32x2_t x =
                __builtin_bit_cast(u32x2_t, __builtin_amdgcn_raw_buffer_load_b64(vt, voff + r * kRow, 0, kPolicy));
            t.v[2 * r] = x[0];
            t.v[2 * r + 1] = x[1];
        } else {
            t.v[r] = __builtin_bit_cast(uint32_t,
                                        __builtin_amdgcn_raw_buffer_load_b32(vt, voff + r * kRow, 0, kPolicy));
        }
    }
    if constexpr (FP8) {
        const float *sp = (lane & 32) ? p.v_scales : p.k_scales;
        t.scl = sp[tile];
    }
}

// Issue the loads of a step: tiles T[u] (a page-head tile index, or the
// complement ~i of one for a tile that is not to be read: past the unit's end
// or in a page outside the pool; its scales are those of tile i) and, `with_q`,
// the unit's query rows. `live` false: a step past the range, nothing is read.
// `blk` < 0: a single-unit step, whose query rows are the group's G heads;
// `blk` >= 0: column block blk of a shared unit (rows 16 blk + n, member r / G
// and head r % G of the group).
template <int D, bool FP8, int NT, bool STREAM>
__device__ __forceinline__ void issue_step(Step<D, FP8, NT> &st, const SplitParams &p, const int32_t (&T)[NT],
                                           bool live, bool with_q, int n, int quad, int lane, int blk)
{
#pragma unroll
    for (int u = 0; u < NT; ++u)
        issue_tile<D, FP8, STREAM>(st.t[u], p, (uint32_t)(T[u] ^ (T[u] >> 31)), live && T[u] >= 0, n, quad, lane);
    const uint32_t row0 = (st.meta >> kMetaUnitShift) * (uint32_t)p.group;
    if (blk < 0) {
        // One tile per step: the q loads are issued only where they read
        // something. Without them in every step the HBM-bound bf16 stream of
        // D = 128 is 0.2% faster; the waits then treat a unit's first step as
        // if its q loads were not there and drain four more loads of the next
        // step once per unit, which costs the others more (D = 64 bf16, 130
        // against 137 us; E4M3 D = 128, 313 against 316).
        if (NT > 1 || with_q)
            load_q<D, FP8>(st.q, p, row0, with_q, n, quad);
    } else if (with_q) {
        // Issued for a unit's first step only: four wavefronts load every tile
        // here, from L2, and with two such workgroups on a CU the load
        // instructions themselves are short. (With loads of zeros in the other
        // steps, a third of them all: 130 prompts of 7030 tokens x 14 samples,
        // 16/1 heads, bf16, D = 128 697 us instead of 619; 16 of 4000 x 24,
        // 12/12 heads, D = 64 155 instead of 126.)
        // Rows past the shared unit's read its first row (never written out).
        const int r = 16 * blk + n, G = p.group;
        const uint32_t rel = r < ((st.valid >> 8) + 1) * G ? (uint32_t)((r / G) * p.num_q_heads + r % G) : 0u;
        const __amdgpu_buffer_rsrc_t qr = buffer_of(p.q + (size_t)row0 * D, 0xffffffffu);
#pragma unroll
        for (int s = 0; s < D / 32; ++s)
            st.q[s] = __builtin_bit_cast(
                u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(
                             qr, (int)(2u * (rel * (uint32_t)D + (uint32_t)q_index<D, FP8>(s, quad))), 0, 0));
    }
}

// Regroup the K tiles (loaded as whole 1 KB runs) into the score-MFMA layout
// through this wave's LDS buffer: lane (t, quad) needs row t, and for bf16
// the 16-byte chunks 4 s + quad (s = 0 .. D/32 - 1), for FP8 the D/64 chunks
// starting at quad D/64. A chunk c of row r is stored at position
// c ^ ((r / P) % C) of its row (P rows per 256 bytes, C chunks per row), which
// makes the 16-lane groups of both the writes and the reads hit distinct banks.
//
// A step's tiles pass through a buffer of one tile in turn: a wave's LDS
// accesses take effect in the order it issues them, so a tile's writes need
// not wait for the reads before them to return. (A buffer for all tiles of a
// step is no faster where LDS is not short, and its 8 or 12 KB more per
// workgroup cost the split and the prefix kernels their second workgroup per
// CU: MI355X, E4M3, D = 128, prefix sharing of 1536 sequences in 768 groups
// 186 us instead of 155; 256 sequences of 1..2048 tokens with 4096 workers 74
// instead of 65. With 4096 sequences in more than 3862 groups the prefix kernel no
// longer fitted a CU at all.)
template <int D, bool FP8, int NT, int N>
__device__ __forceinline__ void regroup_k(const Tile<D, FP8> (&t)[N], uint8_t *lds, int lane, int n, int quad,
                                          u32x4_t (&kc)[NT][FP8 ? D / 64 : D / 32])
{
    constexpr int R = D * (FP8 ? 1 : 2);   // bytes per row
    constexpr int C = R / 16;               // 16-byte chunks per row
    constexpr int P = 256 / R;              // rows per 256 bytes
    const int key = (n / P) % C;
#pragma unroll
    for (int u = 0; u < NT; ++u) {
#pragma unroll
        for (int i = 0; i < Tile<D, FP8>::KW / 4; ++i) {
            const int off = 1024 * i + 16 * lane;
            const int r = off / R, c = (off % R) / 16;
            *reinterpret_cast<u32x4_t *>(lds + r * R + 16 * (c ^ ((r / P) % C))) =
                u32x4_t{t[u].k[4 * i], t[u].k[4 * i + 1], t[u].k[4 * i + 2], t[u].k[4 * i + 3]};
        }
#pragma unroll
        for (int s = 0; s < (FP8 ? D / 64 : D / 32); ++s) {
            const int c = FP8 ? quad * (D / 64) + s : 4 * s + quad;
            kc[u][s] = *reinterpret_cast<const u32x4_t *>(lds + n * R + 16 * (c ^ key));
        }
    }
}

// Score-MFMA A operand for k-step s (8 bf16 values of row t = n).
template <int D, bool FP8>
__device__ __forceinline__ bf16x8_t k_operand(const u32x4_t (&kc)[FP8 ? D / 64 : D / 32], int s)
{
    u32x4_t w;
    if constexpr (!FP8) {
        w = kc[s];
    } else {
        const uint32_t lo = kc[s / 2][2 * (s % 2)], hi = kc[s / 2][2 * (s % 2) + 1];
        uint32_t a, b, c, d;
        e4m3x4_to_bf16(lo, a, b);
        e4m3x4_to_bf16(hi, c, d);
        w = u32x4_t{a, b, c, d};
    }
    return __builtin_bit_cast(bf16x8_t, w);
}

template <int D>
struct Piece {
    f32x4_t acc[D / 16];
    float m;   // running max of this lane's head, base-2 units
    float l;   // this lane's share of the sum of (bf16-rounded) weights
};

template <int D>
__device__ __forceinline__ void reset(Piece<D> &st)
{
#pragma unroll
    for (int i = 0; i < D / 16; ++i)
        st.acc[i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    st.m = kNegInf;
    st.l = 0.f;
}

// One step of the online softmax over the first NT of its tiles. `valid` = live
// tokens of the step (1 .. 16 NT; the first tile has at least one).
//
// With several tiles the score products are independent chains, the running
// maximum is looked at once for all of them, and the value product takes two
// tiles in one v_mfma_f32_16x16x32_bf16 per 16 columns: its k index 8 quad + i
// stands for token 4 quad + (i & 3) of tile i / 4 in both operands, so the
// weights enter exactly as the score MFMAs left them, as with one tile and
// v_mfma_f32_16x16x16bf16_1k.
template <int D, bool FP8, int NT, int N>
__device__ __forceinline__ void compute_step(Piece<D> &st, const Tile<D, FP8> (&t)[N],
                                             const bf16x8_t (&qop)[D / 32], float score_mul, int valid, uint8_t *lds,
                                             int lane, int n, int quad)
{
    static_assert(NT == 1 || NT % 2 == 0, "one tile, or pairs of tiles, per step");
    u32x4_t kc[NT][FP8 ? D / 64 : D / 32];
    regroup_k<D, FP8, NT>(t, lds, lane, n, quad, kc);
    f32x4_t s4[NT];
#pragma unroll
    for (int u = 0; u < NT; ++u)
        s4[u] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < D / 32; ++s)
#pragma unroll
        for (int u = 0; u < NT; ++u)
            s4[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k_operand<D, FP8>(kc[u], s), qop[s], s4[u], 0, 0, 0);

    float vmul[NT];
    float sc[NT][4];
#pragma unroll
    for (int u = 0; u < NT; ++u) {
        float mul = score_mul;
        vmul[u] = 1.0f;
        if constexpr (FP8) {
            const int bits = __builtin_bit_cast(int, t[u].scl);
            mul *= __builtin_bit_cast(float, __builtin_amdgcn_readlane(bits, 0));
            vmul[u] = __builtin_bit_cast(float, __builtin_amdgcn_readlane(bits, 32));
        }
#pragma unroll
        for (int r = 0; r < 4; ++r)
            sc[u][r] = s4[u][r] * mul;
    }
    if (valid < kPageSize * NT) {
#pragma unroll
        for (int u = 0; u < NT; ++u) {
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (kPageSize * u + 4 * quad + r >= valid)
                    sc[u][r] = kNegInf;
            // A missing tile carries the first one's scales: its zero weights must
            // stay zero where that value scale is infinite.
            if (FP8 && kPageSize * u >= valid)
                vmul[u] = 1.0f;
        }
    }
    // The head's maximum over the step (four lanes) is needed only when one of
    // them exceeds the running maximum by the slack: a wave-wide vote skips
    // the cross-lane exchange on the other steps, with the same result.
    float lmx = fmaxf(fmaxf(sc[0][0], sc[0][1]), fmaxf(sc[0][2], sc[0][3]));
#pragma unroll
    for (int u = 1; u < NT; ++u)
        lmx = fmaxf(lmx, fmaxf(fmaxf(sc[u][0], sc[u][1]), fmaxf(sc[u][2], sc[u][3])));
    if (__builtin_amdgcn_ballot_w64(lmx > st.m + kRescaleSlack) != 0) {
        const float mx = quad_max(lmx);
        if (mx > st.m + kRescaleSlack) {
            const float alpha = __builtin_amdgcn_exp2f(st.m - mx);   // 0 on a unit's first tile
            st.l *= alpha;
#pragma unroll
            for (int i = 0; i < D / 16; ++i)
                st.acc[i] *= alpha;
            st.m = mx;
        }
    }
    // The value product takes the weights rounded to bf16, and the sum of
    // weights adds those same rounded values, so the normalisation cancels
    // their rounding: a token that holds all the weight returns its own value
    // row exactly, and the remaining error scales with the spread of the value
    // rows around the output. For E4M3 the weights carry the page's value
    // scale, w = bf16(p s); the sum then adds w / s, the rounded weight without
    // the scale (a zero or non-finite scale, for which that quotient is
    // meaningless, adds the rounded p instead).
    uint32_t pw[NT][2];
#pragma unroll
    for (int u = 0; u < NT; ++u) {
        float pr[4];
#pragma unroll
        for (int r = 0; r < 4; ++r)
            pr[r] = __builtin_amdgcn_exp2f(sc[u][r] - st.m);
        if constexpr (FP8) {
            const uint32_t w01 = pack_bf16(pr[0] * vmul[u], pr[1] * vmul[u]);
            const uint32_t w23 = pack_bf16(pr[2] * vmul[u], pr[3] * vmul[u]);
            pw[u][0] = w01;
            pw[u][1] = w23;
            const float vinv = __builtin_amdgcn_rcpf(vmul[u]);   // wave-uniform
            if (__builtin_isfinite(vinv) && vinv != 0.0f) {
                st.l += ((bf16_lo(w01) + bf16_hi(w01)) + (bf16_lo(w23) + bf16_hi(w23))) * vinv;
            } else {
                const uint32_t p01 = pack_bf16(pr[0], pr[1]);
                const uint32_t p23 = pack_bf16(pr[2], pr[3]);
                st.l += (bf16_lo(p01) + bf16_hi(p01)) + (bf16_lo(p23) + bf16_hi(p23));
            }
        } else {
            const uint32_t p01 = pack_bf16(pr[0], pr[1]);
            const uint32_t p23 = pack_bf16(pr[2], pr[3]);
            st.l += (bf16_lo(p01) + bf16_hi(p01)) + (bf16_lo(p23) + bf16_hi(p23));
            pw[u][0] = p01;
            pw[u][1] = p23;
        }
    }

    // Value operands. Lane (n, quad) holds D/16 consecutive elements of the
    // value rows of tokens 4 quad + r (r = 0..3); value block i takes element i
    // of the four rows, rows 0-1 in its low dword and rows 2-3 in the high one.
    // Byte permutes gather them: bf16 halves directly, E4M3 codes in pairs of
    // rows before one widening per two blocks. Dead slots (only in a
    // sequence's last page) hold arbitrary cache contents and are zeroed first,
    // as 0 * NaN would poison the MFMA.
    constexpr int VR = Tile<D, FP8>::VW / 4;   // dwords per row
    uint32_t vr[NT][4 * VR];
#pragma unroll
    for (int u = 0; u < NT; ++u)
#pragma unroll
        for (int k = 0; k < 4 * VR; ++k)
            vr[u][k] = t[u].v[k];
    if (valid < kPageSize * NT) {
#pragma unroll
        for (int u = 0; u < NT; ++u)
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int c = 0; c < VR; ++c)
                    vr[u][r * VR + c] = kPageSize * u + 4 * quad + r < valid ? vr[u][r * VR + c] : 0u;
    }
#pragma unroll
    for (int i = 0; i < D / 16; i += 2) {
        uint32_t a0[2 * NT], a1[2 * NT];   // operands of blocks i and i + 1
#pragma unroll
        for (int u = 0; u < NT; ++u) {
            if constexpr (FP8) {
                // Bytes (row a, row b) of elements i and i + 1, then one widening per element.
                const int c = i / 4;
                const uint32_t sel = (i % 4) == 0 ? 0x05010400u : 0x07030602u;
                const uint32_t p01 = __builtin_amdgcn_perm(vr[u][VR + c], vr[u][c], sel);
                const uint32_t p23 = __builtin_amdgcn_perm(vr[u][3 * VR + c], vr[u][2 * VR + c], sel);
                a0[2 * u] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(p01, 1.0f, false));
                a1[2 * u] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(p01, 1.0f, true));
                a0[2 * u + 1] =
                    __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(p23, 1.0f, false));
                a1[2 * u + 1] =
                    __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(p23, 1.0f, true));
            } else {
                // Dword w holds elements 2w (low half) and 2w + 1 (high half) of a row.
                const int w = i / 2;
                a0[2 * u] = __builtin_amdgcn_perm(vr[u][VR + w], vr[u][w], 0x05040100u);
                a1[2 * u] = __builtin_amdgcn_perm(vr[u][VR + w], vr[u][w], 0x07060302u);
                a0[2 * u + 1] = __builtin_amdgcn_perm(vr[u][3 * VR + w], vr[u][2 * VR + w], 0x05040100u);
                a1[2 * u + 1] = __builtin_amdgcn_perm(vr[u][3 * VR + w], vr[u][2 * VR + w], 0x07060302u);
            }
        }
        if constexpr (NT > 1) {
#pragma unroll
            for (int h = 0; h < NT; h += 2) {
                const bf16x8_t b =
                    __builtin_bit_cast(bf16x8_t, u32x4_t{pw[h][0], pw[h][1], pw[h + 1][0], pw[h + 1][1]});
                st.acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                    __builtin_bit_cast(bf16x8_t, u32x4_t{a0[2 * h], a0[2 * h + 1], a0[2 * h + 2], a0[2 * h + 3]}), b,
                    st.acc[i], 0, 0, 0);
                st.acc[i + 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                    __builtin_bit_cast(bf16x8_t, u32x4_t{a1[2 * h], a1[2 * h + 1], a1[2 * h + 2], a1[2 * h + 3]}), b,
                    st.acc[i + 1], 0, 0, 0);
            }
        } else {
            const i16x4_t b = __builtin_bit_cast(i16x4_t, u32x2_t{pw[0][0], pw[0][1]});
            st.acc[i] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(
                __builtin_bit_cast(i16x4_t, u32x2_t{a0[0], a0[1]}), b, st.acc[i], 0, 0, 0);
            st.acc[i + 1] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(
                __builtin_bit_cast(i16x4_t, u32x2_t{a1[0], a1[1]}), b, st.acc[i + 1], 0, 0, 0);
        }
    }
}

// Store this lane's share of a partial state (m, l, acc) as row `row` of
// (part_ml [][2], part_acc [][D]); l is the head's full sum (quad_sum).
template <int D>
__device__ __forceinline__ void store_partial(const Piece<D> &st, float l, bool bad, float *part_ml,
                                              float *part_acc, size_t row, int quad)
{
    const float poison = bad ? __builtin_nanf("") : 0.0f;
    float *dst = part_acc + row * D + quad * (D / 4);
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int i = 0; i < D / 16; i += 4)
            *reinterpret_cast<f32x4_t *>(dst + r * (D / 16) + i) =
                f32x4_t{st.acc[i][r], st.acc[i + 1][r], st.acc[i + 2][r], st.acc[i + 3][r]} + poison;
    if (quad == 0)   // a NaN maximum keeps the poison alive through the merge weights
        *reinterpret_cast<f32x2_t *>(part_ml + row * 2) = f32x2_t{st.m + poison, l};
}

// Finish the current unit: normalise and write its bf16 rows if the whole unit
// was seen and nothing else is merged into it (`full`), else store the partial
// state, G rows, in slot `slot` of (part_ml, part_acc).
template <int D>
__device__ __forceinline__ void finish_unit(const SplitParams &p, Piece<D> &st, uint32_t row0, bool full,
                                            bool bad, float *part_ml, float *part_acc, size_t slot, int n,
                                            int quad)
{
    const int G = p.group;
    const float l = quad_sum(st.l);
    const int d0 = quad * (D / 4);   // this lane holds O[row0 + n][d0 .. d0 + D/4)
    if (n >= G)
        return;
    if (full) {
        const float inv = bad ? __builtin_nanf("") : 1.0f / l;
        uint8_t *dst = reinterpret_cast<uint8_t *>(p.out + ((size_t)row0 + n) * D + d0);
#pragma unroll
        for (int c = 0; c < D / 32; ++c) {
            // output columns d0 + 8c .. 8c + 7 are acc[i][r] with r * D/16 + i = 8c + ...
            uint32_t wv[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int k0 = 8 * c + 2 * e;   // flat index r * (D/16) + i
                const int r0 = k0 / (D / 16), i0 = k0 % (D / 16);
                const int k1 = k0 + 1;
                const int r1 = k1 / (D / 16), i1 = k1 % (D / 16);
                wv[e] = pack_bf16(st.acc[i0][r0] * inv, st.acc[i1][r1] * inv);
            }
            *reinterpret_cast<u32x4_t *>(dst + 16 * c) = u32x4_t{wv[0], wv[1], wv[2], wv[3]};
        }
    } else {
        store_partial<D>(st, l, bad, part_ml, part_acc, slot * G + n, quad);
    }
}

struct ScanSum {
    static constexpr int32_t kIdentity = 0;
    __device__ static int32_t op(int32_t a, int32_t b) { return a + b; }
};
struct ScanMax {
    static constexpr int32_t kIdentity = -2147483647 - 1;
    __device__ static int32_t op(int32_t a, int32_t b) { return a > b ? a : b; }
};

// Output staging for plain attention. Vector-memory stores and loads share
// one completion counter on this part, so a wait for a load issued after a
// store also waits for the store, which under a full read stream takes
// microseconds: writing each finished unit's rows out at once stalled the
// worker at its next tile (measured: ~2.9 us per unit with 256-token
// sequences), and so did the partial state of the range's first, cut unit
// (2.6% of the 7B-like step). Finished rows are therefore normalised into a
// per-wave LDS stage, and the first piece's state kept there too, and both
// are written out only when the stage is full or the worker's range ends,
// where no later load waits on them.
constexpr int kOutStageBytes = 16384;                       // per wave
constexpr int kMaxOutSlots = kOutStageBytes / (1 * 64 * 2); // smallest slot: G = 1, D = 64

// The bf16 rows of a finished unit (this lane's D/4 outputs of row n) into
// its stage slot; l is the head's full sum of weights.
template <int D>
__device__ __forceinline__ void stage_output(const Piece<D> &st, float l, bool bad, uint8_t *slot, int n, int quad)
{
    const float inv = bad ? __builtin_nanf("") : 1.0f / l;
    uint8_t *dst = slot + ((size_t)n * D + quad * (D / 4)) * 2;
#pragma unroll
    for (int c = 0; c < D / 32; ++c) {
        uint32_t wv[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int k0 = 8 * c + 2 * e;   // flat index r * (D/16) + i, as in finish_unit
            const int r0 = k0 / (D / 16), i0 = k0 % (D / 16);
            const int k1 = k0 + 1;
            const int r1 = k1 / (D / 16), i1 = k1 % (D / 16);
            wv[e] = pack_bf16(st.acc[i0][r0] * inv, st.acc[i1][r1] * inv);
        }
        *reinterpret_cast<u32x4_t *>(dst + 16 * c) = u32x4_t{wv[0], wv[1], wv[2], wv[3]};
    }
}

// Write the first `count` staged units out. A unit's G rows are one
// contiguous block of G * D * 2 bytes both in the stage and in `out` (from
// row rows[s]), so every lane copies 16-byte pieces 1 KB apart: each store
// instruction writes whole cache lines. (Stored straight from the
// accumulator layout, each instruction left 16-byte pieces 64 bytes apart,
// over a hundred partial-line writes per unit, which drained slowly enough
// under a full read stream to cost ~20 us per flush of nine units.)
__device__ __forceinline__ void flush_outputs(const SplitParams &p, int head_dim, const uint8_t *stage,
                                              const uint32_t *rows, int count, int slot_bytes, int lane)
{
    for (int s = 0; s < count; ++s) {
        const uint8_t *src = stage + (size_t)s * slot_bytes;
        uint8_t *dst = reinterpret_cast<uint8_t *>(p.out + (size_t)rows[s] * head_dim);
        for (int off = 16 * lane; off < slot_bytes; off += 16 * kWave)
            *reinterpret_cast<u32x4_t *>(dst + off) = *reinterpret_cast<const u32x4_t *>(src + off);
    }
}

// The partial state (m, l, acc) of a cut unit into the stage, laid out as
// in the workspace: G rows of D fp32 (acc), then G pairs (m, l); l is the
// head's full sum of weights.
template <int D>
__device__ __forceinline__ void stage_partial(const Piece<D> &st, float l, bool bad, uint8_t *area, int G, int n,
                                              int quad)
{
    const float poison = bad ? __builtin_nanf("") : 0.0f;
    float *acc = reinterpret_cast<float *>(area) + (size_t)n * D + quad * (D / 4);
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int i = 0; i < D / 16; i += 4)
            *reinterpret_cast<f32x4_t *>(acc + r * (D / 16) + i) =
                f32x4_t{st.acc[i][r], st.acc[i + 1][r], st.acc[i + 2][r], st.acc[i + 3][r]} + poison;
    if (quad == 0)
        *reinterpret_cast<f32x2_t *>(reinterpret_cast<float *>(area) + (size_t)G * D + 2 * n) =
            f32x2_t{st.m + poison, l};
}

// Write a staged partial state to slot `slot` of (part_ml, part_acc) as two
// contiguous blocks.
__device__ __forceinline__ void flush_partial(const SplitParams &p, int head_dim, const uint8_t *area, size_t slot,
                                              int lane)
{
    const int G = p.group;
    const int acc_bytes = G * head_dim * 4;
    uint8_t *dst = reinterpret_cast<uint8_t *>(p.part_acc + slot * G * head_dim);
    for (int off = 16 * lane; off < acc_bytes; off += 16 * kWave)
        *reinterpret_cast<u32x4_t *>(dst + off) = *reinterpret_cast<const u32x4_t *>(area + off);
    if (lane < G)
        *reinterpret_cast<f32x2_t *>(p.part_ml + (slot * G + lane) * 2) =
            *reinterpret_cast<const f32x2_t *>(area + acc_bytes + 8 * lane);
}

// Prefix own pages: the fp32 states of finished own units that the merge
// combines are queued per wave in LDS and written when the queue is full or
// the range ends, for the reason given above for the output stage. The queue
// holds two states at G <= 8 (D = 128) and stays small, so the fused prefix
// kernel keeps two workgroups per CU (a 16 KB queue per wave did not).
constexpr int kOwnStageBytes = 8448;                        // per wave
constexpr int kMaxOwnSlots = kOwnStageBytes / ((1 * (64 + 2) * 4 + 15) & ~15);

// The workgroup's queues, one per wave. Idle until its workers start: the
// prefix kernel keeps the groups' description here while it derives the streams.
__device__ __forceinline__ uint8_t *own_state_stage()
{
    __shared__ __attribute__((aligned(16))) uint8_t own_stage[kWavesPerBlock * kOwnStageBytes];
    return own_stage;
}

// Write `count` queued states: entry s holds G rows of D fp32 (acc) and G
// pairs (m, l) as stage_partial lays them out; dest[s] = slot << 1 | (unit
// area ? 1 : 0), the slot in (part_ml, part_acc) or (unit_ml, unit_acc).
__device__ __forceinline__ void flush_states(const SplitParams &p, int head_dim, const uint8_t *stage,
                                             const uint32_t *dest, int count, int area_bytes, int lane)
{
    const int G = p.group;
    const int acc_bytes = G * head_dim * 4;
    for (int s = 0; s < count; ++s) {
        const uint32_t d = dest[s];
        const size_t slot = d >> 1;
        float *const pml = (d & 1u) ? p.unit_ml : p.part_ml;
        float *const pacc = (d & 1u) ? p.unit_acc : p.part_acc;
        const uint8_t *area = stage + (size_t)s * area_bytes;
        uint8_t *dst = reinterpret_cast<uint8_t *>(pacc + slot * G * head_dim);
        for (int off = 16 * lane; off < acc_bytes; off += 16 * kWave)
            *reinterpret_cast<u32x4_t *>(dst + off) = *reinterpret_cast<const u32x4_t *>(area + off);
        if (lane < G)
            *reinterpret_cast<f32x2_t *>(pml + (slot * G + lane) * 2) =
                *reinterpret_cast<const f32x2_t *>(area + acc_bytes + 8 * lane);
    }
}

// One array's part of a workgroup scan: the thread's contiguous run of a[0, n)
// and, after wave(), its exclusive prefix within the wavefront. (DPP scans: as
// shuffles, each of the six steps is a round trip through LDS.)
template <class Op>
struct RunScan {
    int32_t *a;
    int lo, hi, excl;

    // The run's place and the wavefront's scan; lane 63 leaves the wavefront's total in *total.
    __device__ __forceinline__ void wave(int32_t *arr, int n, int32_t *total)
    {
        constexpr int T = kWave * kWavesPerBlock;
        const int tid = threadIdx.x, per = (n + T - 1) / T;
        a = arr;
        lo = min(n, tid * per);
        hi = min(n, lo + per);
        int local = Op::kIdentity;
        for (int i = lo; i < hi; ++i)
            local = Op::op(local, a[i]);
        const int incl = wave_scan<Op>(local);
        excl = lane_from<0x138, 0xf>(incl, Op::kIdentity);   // the lane before's
        if ((tid & (kWave - 1)) == kWave - 1)
            *total = incl;
    }
    // Writes the run's exclusive prefixes; returns the total of all wavefronts.
    __device__ __forceinline__ int finish(const int32_t *totals) const
    {
        const int wave = threadIdx.x / kWave;
        int run = excl, total = Op::kIdentity;
#pragma unroll
        for (int k = 0; k < kWavesPerBlock; ++k) {
            if (k < wave)
                run = Op::op(run, totals[k]);
            total = Op::op(total, totals[k]);
        }
        for (int i = lo; i < hi; ++i) {
            const int v = a[i];
            a[i] = run;
            run = Op::op(run, v);
        }
        return total;
    }
};

// Turns a[0, n) (in LDS, written before a barrier) into its exclusive
// prefix scan under Op (sum or maximum) and stores the total in a[n]. Every
// thread of the workgroup calls it; each scans a contiguous run. Ends with a
// barrier.
template <class Op = ScanSum>
__device__ __forceinline__ void block_exclusive_scan(int32_t *a, int n)
{
    __shared__ int32_t s_wave[kWavesPerBlock];
    RunScan<Op> sa;
    sa.wave(a, n, s_wave + threadIdx.x / kWave);
    __syncthreads();
    const int total = sa.finish(s_wave);
    if (threadIdx.x == 0)
        a[n] = total;
    __syncthreads();
}

// Two independent exclusive scans, a[0, n) under OpA and b[0, m) under OpB,
// with their totals in a[n] and b[m], sharing the barriers of one scan.
template <class OpA, class OpB>
__device__ __forceinline__ void block_exclusive_scan2(int32_t *a, int n, int32_t *b, int m)
{
    __shared__ int32_t s_wave[2][kWavesPerBlock];
    RunScan<OpA> sa;
    RunScan<OpB> sb;
    sa.wave(a, n, s_wave[0] + threadIdx.x / kWave);
    sb.wave(b, m, s_wave[1] + threadIdx.x / kWave);
    __syncthreads();
    const int tot_a = sa.finish(s_wave[0]), tot_b = sb.finish(s_wave[1]);
    if (threadIdx.x == 0) {
        a[n] = tot_a;
        b[m] = tot_b;
    }
    __syncthreads();
}

// floor(x / y) for 0 <= x < 2^16, 0 < y < 2^13: (x + 1/2) / y is at least
// 1 / 2y away from every integer, far more than the reciprocal's error. (An
// integer division is some 30 dependent instructions, 0.1 us.)
__device__ __forceinline__ int small_div(int x, int y)
{
    return (int)(((float)x + 0.5f) * __builtin_amdgcn_rcpf((float)y));
}

// Pages of a sequence of length L: ceil(clamp(L, 0, max_len) / 16).
__device__ __forceinline__ int pages_of(int L, int max_len)
{
    return L <= 0 ? 0 : (min(L, max_len) + kPageSize - 1) / kPageSize;
}

// Plain attention, run by the whole workgroup before its workers start: the
// steps (of NT pages) per sequence and KV head, their exclusive prefix sum in
// s_cum[0 .. B] and the lengths in s_len[0 .. B), all in LDS; workgroup 0 also
// stores the prefix sum for the merge.
template <int NT>
__device__ __forceinline__ void scan_sequences(const SplitParams &p, int32_t *s_cum, int32_t *s_len)
{
    constexpr int T = kWave * kWavesPerBlock;
    const int B = p.batch;
    const int max_len = p.max_blocks * kPageSize;
    for (int b = threadIdx.x; b < B; b += T) {
        const int L = p.seq_lens[b];
        s_len[b] = L;
        s_cum[b] = (pages_of(L, max_len) + NT - 1) / NT;
    }
    __syncthreads();
    block_exclusive_scan(s_cum, B);
    if (blockIdx.x == 0)
        for (int b = threadIdx.x; b <= B; b += T)
            p.cum_out[b] = s_cum[b];
}

// This wave's staging area for regrouping K tiles (16 tokens x D elements).
// Declared here, keyed only on the tile shape, so that a kernel running the
// worker in several modes (prefix sharing: own and shared pages in different
// workgroups) holds one such array, not one per mode.
template <int D, bool FP8>
__device__ __forceinline__ uint8_t *k_regroup_stage()
{
    __shared__ __attribute__((aligned(16)))
    uint8_t k_stage[kWavesPerBlock][kPageSize * D * (FP8 ? 1 : 2)];
    return k_stage[__builtin_amdgcn_readfirstlane(threadIdx.x / kWave)];
}

// Which tiles a worker streams.
constexpr int kAllPages = 0;      // plain attention: every page of every sequence
constexpr int kOwnPages = 1;      // prefix sharing: the pages after each sequence's shared ones
constexpr int kSharedPages = 2;   // prefix sharing: each group's shared pages once, one column block per wavefront

// LDS view of the unit stream: the exclusive prefix sum of steps per sequence
// and KV head, and the lengths; for kOwnPages also each sequence's shared pages
// (its own pages start after them). For kSharedPages the "sequences" are the
// sub-groups: `cum` is their prefix sum of shared steps and `gl` packs each
// one's first member, size and the tiles missing from its last step:
// lead | (members - 1) << 16 | missing << 24.
struct StreamLds {
    const int32_t *cum;     // [B + 1], or [S + 1] for kSharedPages
    const int32_t *len;     // [B]
    const int32_t *shared;  // [B], kOwnPages only
    const int32_t *gl;      // [S], kSharedPages only
    int32_t num_groups;     // S, kSharedPages only
};

// Worker w of the split-KV pass over the stream that `sv` describes (in LDS,
// complete: the caller has passed a barrier). A worker is one wavefront, or
// for kSharedPages the four wavefronts of a workgroup, which stream the same
// tiles and compute column blocks blk = 0..3 of each shared unit.
template <int D, bool FP8, int MODE>
__device__ __forceinline__ void split_unit_worker(const SplitParams &p, int w, const StreamLds &sv, int blk = -1)
{
    constexpr bool kShared = MODE == kSharedPages;
    constexpr int kNbuf = kPipelineDepth;
    if (w >= p.num_workers)
        return;
    const int nseq = kShared ? sv.num_groups : p.batch;   // "sequences" of the stream
    constexpr int NT = step_tiles<D, FP8>();
    const int Hkv = p.num_kv_heads;
    const long long total = (long long)sv.cum[nseq] * Hkv;
    const int nw = effective_workers(total, p.num_workers, NT, kShared ? 0 : wide_from(p.num_workers, FP8));
    if (w >= nw)
        return;
    const int s0 = __builtin_amdgcn_readfirstlane((int)((long long)w * total / nw));
    const int nsteps = __builtin_amdgcn_readfirstlane((int)((long long)(w + 1) * total / nw)) - s0;
    if (nsteps <= 0)
        return;
    const int lane = threadIdx.x & (kWave - 1);
    const int n = lane & 15;
    const int quad = lane >> 4;
    const int G = p.group;
    uint8_t *lds = k_regroup_stage<D, FP8>();
    // Plain attention: a per-wave stage (see stage_output) holding the
    // partial state of the range's first piece, if cut (G * (D + 2) fp32 at
    // the start), then the output rows of finished units, `staged` of them
    // queued, each slot G rows of D bf16.
    constexpr bool kStageOut = MODE == kAllPages;
    __shared__ uint8_t out_stage[kWavesPerBlock][kStageOut ? kOutStageBytes : 16];
    __shared__ uint32_t out_rows[kWavesPerBlock][kStageOut ? kMaxOutSlots : 1];
    uint8_t *const ostage_base = out_stage[__builtin_amdgcn_readfirstlane(threadIdx.x / kWave)];
    uint32_t *const orows = out_rows[__builtin_amdgcn_readfirstlane(threadIdx.x / kWave)];
    const int part_bytes = (G * (D + 2) * 4 + 15) & ~15;   // keeps the output slots 16-byte aligned
    uint8_t *const ostage = ostage_base + part_bytes;
    const int slot_bytes = G * D * 2;
    const int out_slots = (kOutStageBytes - part_bytes) / slot_bytes;   // >= 1 (G <= 16, D <= 128)
    int staged = 0;
    bool part_staged = false;
    // Prefix own pages: the queue of finished own units' states (flush_states).
    constexpr bool kStageOwn = MODE == kOwnPages;
    __shared__ uint32_t own_dest[kWavesPerBlock][kStageOwn ? kMaxOwnSlots : 1];
    uint8_t *qstage = nullptr;
    if constexpr (kStageOwn)
        qstage = own_state_stage() + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave) * kOwnStageBytes;
    uint32_t *const qdest = own_dest[__builtin_amdgcn_readfirstlane(threadIdx.x / kWave)];
    const int own_slots = kStageOwn ? kOwnStageBytes / part_bytes : 0;   // 1 or more (G <= 16, D <= 128)
    int queued = 0;

    // Step descriptors, a chunk of kChunk steps at a time, one step per lane:
    // lane i finds the unit and the pages of its step in the stream and loads
    // their block-table entries; the streaming loop then only reads lanes. Per
    // step that costs two or three lane reads instead of a cursor's compares,
    // selects and table loads, which at one wavefront per SIMD are time that
    // nothing else fills. A chunk's table entries are loaded while the chunk
    // before it streams.
    constexpr int kChunk = kWave / kNbuf * kNbuf;
    const __amdgpu_buffer_rsrc_t btab =
        buffer_of(p.block_table, (uint32_t)(p.batch * p.max_blocks) * (uint32_t)sizeof(int32_t));
    const int max_len = p.max_blocks * kPageSize;
    const int top = nseq > 1 ? 1 << (31 - __builtin_clz((unsigned)nseq - 1)) : 0;   // largest power of two below nseq
    struct Desc {
        int32_t bt[NT];       // block-table entries (in flight)
        uint32_t meta;
        int32_t valid, tiles, g;
    };
    auto find = [&](int c0) -> Desc {   // the descriptor of step s0 + c0 + lane (the range's last one past its end)
        const uint32_t x = (uint32_t)(s0 + min(c0 + lane, nsteps - 1));
        const int xq = (int)(x / (uint32_t)Hkv);
        int b = 0;   // largest b with Hkv cum[b] <= x (its steps are not empty)
        for (int half = top; half > 0; half >>= 1)
            if (b + half < nseq && sv.cum[b + half] <= xq)
                b += half;
        const int first = sv.cum[b], steps = sv.cum[b + 1] - first;
        const uint32_t off = x - (uint32_t)first * (uint32_t)Hkv;
        const int g = (int)(off / (uint32_t)steps), j = (int)(off - (uint32_t)g * (uint32_t)steps);
        Desc d;
        int row, page;
        if constexpr (kShared) {   // read through the sub-group's first member's row; every shared page is full
            const int gl = sv.gl[b];
            row = gl & 0xffff;
            page = j * NT;
            d.tiles = j == steps - 1 ? NT - (gl >> 24) : NT;
            d.valid = kPageSize * d.tiles | ((gl >> 16) & 15) << 8;
            d.meta = 0;
        } else {
            const int len = sv.len[b];
            const int sh = MODE == kOwnPages ? sv.shared[b] : 0;
            row = b;
            page = sh + j * NT;
            d.tiles = min(NT, pages_of(len, max_len) - page);
            d.valid = max(1, min(kPageSize * d.tiles, len - page * kPageSize));
            d.meta = (len > max_len ? kMetaBad : 0u) | (sh > 0 ? kMetaPrefixed : 0u);
        }
        d.g = g;
        d.meta |= (uint32_t)(row * Hkv + g) << kMetaUnitShift | (j == 0 ? kMetaFirst : 0u) |
                  (j == steps - 1 ? kMetaLast : 0u);
#pragma unroll
        for (int u = 0; u < NT; ++u)
            d.bt[u] = (int32_t)__builtin_amdgcn_raw_buffer_load_b32(btab, 4 * (row * p.max_blocks + page + u), 0, 0);
        return d;
    };
    int32_t tile[NT];     // per lane: issue_step's T of the lane's step
    uint32_t lmeta;       // its metadata (kMetaBad also for a page outside the pool)
    int32_t lvalid;
    auto settle = [&](const Desc &d) {
        bool bad = false;
#pragma unroll
        for (int u = 0; u < NT; ++u) {
            const bool in = (uint32_t)d.bt[u] < (uint32_t)p.num_pages, has = u < d.tiles;
            const int32_t at = d.bt[u] * Hkv + d.g;
            tile[u] = has && in ? at : ~(u > 0 ? tile[0] ^ (tile[0] >> 31) : 0);
            bad |= has && !in;
        }
        lmeta = d.meta | (bad ? kMetaBad : 0u);
        lvalid = d.valid;
    };
    int cpos = 0, cnext = kChunk;   // lane of the next step to issue; first step of the chunk in `ahead`
    Desc ahead = find(0);
    settle(ahead);
    auto issue = [&](Step<D, FP8, NT> &x, int i, bool with_q) {   // step i of the range, from lane cpos
        int32_t T[NT];
#pragma unroll
        for (int u = 0; u < NT; ++u)
            T[u] = __builtin_amdgcn_readlane(tile[u], cpos);
        x.meta = (uint32_t)__builtin_amdgcn_readlane((int)lmeta, cpos);
        x.valid = __builtin_amdgcn_readlane(lvalid, cpos);
        issue_step<D, FP8, NT, !kShared>(x, p, T, i < nsteps, with_q || (x.meta & kMetaFirst) != 0, n, quad, lane, blk);
        ++cpos;
    };

    Step<D, FP8, NT> buf[kNbuf];
#pragma unroll
    for (int k = 0; k < kNbuf - 1; ++k)
        issue(buf[k], k, k == 0);
    // (after the first loads: the search takes about as long as they do)
    if (nsteps > kChunk)
        ahead = find(kChunk);

    Piece<D> st;
    reset(st);
    bf16x8_t qop[D / 32];   // score-MFMA B operands of the current unit (zero columns past its rows)
    bool started = false;   // the current unit's first tile is inside this range
    bool bad = false;
    int slot_sel = 0;
    for (int i0 = 0; i0 < nsteps; i0 += kNbuf) {
#pragma unroll
        for (int k = 0; k < kNbuf; ++k) {
            const int i = i0 + k;
            if (k == 1 && cpos == kChunk) {   // (the step issued at k == 1 is a multiple of kNbuf)
                settle(ahead);
                cpos = 0;
                cnext += kChunk;
                if (cnext < nsteps)
                    ahead = find(cnext);
            }
            issue(buf[(k + kNbuf - 1) % kNbuf], i + kNbuf - 1, false);
            if (i < nsteps) {
                const Step<D, FP8, NT> &t = buf[k];
                const uint32_t meta = t.meta;
                const bool ends = i == nsteps - 1;
                if (i == 0 || (meta & kMetaFirst) != 0) {
#pragma unroll
                    for (int s = 0; s < D / 32; ++s)
                        qop[s] = __builtin_bit_cast(bf16x8_t, t.q[s]);
                }
                started |= (meta & kMetaFirst) != 0;
                bad |= (meta & kMetaBad) != 0;
                // Of a step of four tiles a short unit has one or two, and the others would
                // cost as much; only a unit's last step can lack any. E4M3, D = 64, MI355X,
                // four tiles -> those that there are: 5663 sequences of one page, 3/3
                // heads, 45.5 -> 37.0 us (steps of one tile 36.4); 8192, 8/2 heads,
                // 62.0 -> 54.3; of 3 or 4 pages 32.6 -> 33.7 (38.4 to 42.6); longer ones the
                // same. (With the choice in every step those took 1% longer. Shared units
                // are long: their loop lost 5%.)
                constexpr bool kFew = NT == 4 && !kShared;
                const int valid = kShared ? t.valid & 0xff : t.valid;
                if (kFew && (meta & kMetaLast) == 0)
                    compute_step<D, FP8, NT>(st, t.t, qop, p.scale_log2, kPageSize * NT, lds, lane, n, quad);
                else if (kFew && valid <= kPageSize)
                    compute_step<D, FP8, 1>(st, t.t, qop, p.scale_log2, valid, lds, lane, n, quad);
                else if (kFew && valid <= 2 * kPageSize)
                    compute_step<D, FP8, 2>(st, t.t, qop, p.scale_log2, valid, lds, lane, n, quad);
                else
                    compute_step<D, FP8, NT>(st, t.t, qop, p.scale_log2, valid, lds, lane, n, quad);
                if (kShared && ((meta & kMetaLast) != 0 || ends)) {
                    // A shared unit's state is always merged: a whole one goes to the unit area
                    // (indexed by first query row / G), a cut one to the worker's slot; block blk
                    // holds rows 16 blk .. 16 blk + 15 of the unit's kPrefixRows.
                    const uint32_t unit = meta >> kMetaUnitShift;
                    const bool whole = started && (meta & kMetaLast) != 0;
                    const size_t slot = whole ? (size_t)unit : 2 * (size_t)w + slot_sel;
                    const int r = 16 * blk + n;
                    const float l = quad_sum(st.l);
                    if (r < ((t.valid >> 8) + 1) * G)
                        store_partial<D>(st, l, bad, whole ? p.unit_ml : p.part_ml, whole ? p.unit_acc : p.part_acc,
                                         slot * kPrefixRows + r, quad);
                    reset(st);
                    started = false;
                    bad = false;
                    slot_sel = 1;
                } else if (!kShared && ((meta & kMetaLast) != 0 || ends)) {
                    // A unit cut by this range leaves its piece in the worker's slot 2w + slot_sel.
                    // A whole unit is written out, unless it still has to be merged (shared pages,
                    // or the own pages of a sequence that has them): then its state goes to its
                    // own slot in the unit area, indexed by (first query row) / G.
                    const uint32_t unit = meta >> kMetaUnitShift, row0 = unit * (uint32_t)G;
                    const bool whole = started && (meta & kMetaLast) != 0;
                    const bool to_unit = whole && (meta & kMetaPrefixed) != 0;
                    float *const pml = to_unit ? p.unit_ml : p.part_ml;
                    float *const pacc = to_unit ? p.unit_acc : p.part_acc;
                    const size_t slot = to_unit ? (size_t)unit : 2 * (size_t)w + slot_sel;
                    if (kStageOut && whole) {
                        const float l = quad_sum(st.l);
                        if (n < G)
                            stage_output<D>(st, l, bad, ostage + (size_t)staged * slot_bytes, n, quad);
                        if (lane == 0)
                            orows[staged] = row0;
                        if (++staged == out_slots) {
                            flush_outputs(p, D, ostage, orows, staged, slot_bytes, lane);
                            staged = 0;
                        }
                    } else if (kStageOut && slot_sel == 0) {
                        // the range's first piece, cut: written out with the stage at the end
                        const float l = quad_sum(st.l);
                        if (n < G)
                            stage_partial<D>(st, l, bad, ostage_base, G, n, quad);
                        part_staged = true;
                    } else if (kStageOwn && !(whole && !to_unit)) {
                        // a state the merge combines: queued
                        const float l = quad_sum(st.l);
                        if (queued == own_slots) {
                            flush_states(p, D, qstage, qdest, queued, part_bytes, lane);
                            queued = 0;
                        }
                        if (n < G)
                            stage_partial<D>(st, l, bad, qstage + (size_t)queued * part_bytes, G, n, quad);
                        if (lane == 0)
                            qdest[queued] = (uint32_t)(slot << 1) | (to_unit ? 1u : 0u);
                        ++queued;
                    } else {
                        finish_unit<D>(p, st, row0, whole && !to_unit, bad, pml, pacc, slot, n, quad);
                    }
                    reset(st);
                    started = false;
                    bad = false;
                    slot_sel = 1;
                }
            }
        }
    }
    if (kStageOut && staged > 0)
        flush_outputs(p, D, ostage, orows, staged, slot_bytes, lane);
    if (kStageOut && part_staged)
        flush_partial(p, D, ostage_base, 2 * (size_t)w, lane);
    if (kStageOwn && queued > 0)
        flush_states(p, D, qstage, qdest, queued, part_bytes, lane);
}

}  // namespace
}  // namespace sl

#endif  // SL_DECODE_UNIT_H
