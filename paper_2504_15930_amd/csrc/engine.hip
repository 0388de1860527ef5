// Device code of the decode engine (engine.cpp): filling newly admitted
// prompts' pages with synthetic key/value data, and the one-launch step for
// steps with little attention work. (Otherwise a step's bookkeeping is
// applied by the KV-append launch, append.hip, or by the merge launch.)
#include "append_unit.h"
#include "decode_unit.h"
#include "engine_internal.h"

namespace sl {
namespace {

constexpr int kEngineThreads = 256;

// 32-bit integer mixer ("lowbias32": xorshift-multiply rounds).
__device__ __forceinline__ uint32_t mix32(uint32_t x)
{
    x ^= x >> 16;
    x *= 0x7feb352du;
    x ^= x >> 15;
    x *= 0x846ca68bu;
    x ^= x >> 16;
    return x;
}

// One workgroup per (prompt page, KV head) tile: 16 x D synthetic values for
// K and V. bf16: uniform in [-2, 2). E4M3: codes of magnitude below 2 (exponent
// field <= 7) with a random sign, and scale 1.
template <int D, bool FP8>
__global__ __launch_bounds__(kEngineThreads) void engine_fill_kernel(const int32_t *pages, int32_t hkv,
                                                                     uint32_t seed, void *k_pages, void *v_pages,
                                                                     float *k_scales, float *v_scales)
{
    const int page = pages[blockIdx.x / hkv];
    const int g = blockIdx.x % hkv;
    const size_t tile = (size_t)page * hkv + g;
    const uint32_t base = seed ^ ((uint32_t)tile * 0x9e3779b1u);
    for (int e = threadIdx.x; e < kPageSize * D; e += kEngineThreads) {
        const uint32_t hk = mix32(base ^ ((uint32_t)e * 0x85ebca77u));
        const uint32_t hv = mix32(hk ^ 0xc2b2ae3du);
        if constexpr (FP8) {
            static_cast<uint8_t *>(k_pages)[tile * kPageSize * D + e] = (uint8_t)((hk & 0x3fu) | ((hk >> 24) & 0x80u));
            static_cast<uint8_t *>(v_pages)[tile * kPageSize * D + e] = (uint8_t)((hv & 0x3fu) | ((hv >> 24) & 0x80u));
        } else {
            const float fk = ((float)(hk >> 8) * (1.0f / 16777216.0f) - 0.5f) * 4.0f;
            const float fv = ((float)(hv >> 8) * (1.0f / 16777216.0f) - 0.5f) * 4.0f;
            static_cast<__bf16 *>(k_pages)[tile * kPageSize * D + e] = (__bf16)fk;
            static_cast<__bf16 *>(v_pages)[tile * kPageSize * D + e] = (__bf16)fv;
        }
    }
    if constexpr (FP8) {
        if (threadIdx.x == 0) {
            k_scales[tile] = 1.0f;
            v_scales[tile] = 1.0f;
        }
    }
}

// ---------------------------------------------------------------------------
// One-launch step (UnitStepParams). Workgroups, in this order:
//   unit_blocks  attention: K_e workgroups per unit (sequence e, KV head g);
//                the unit's tiles are split evenly over its K_e * kUnitWaves
//                waves, each running the split kernel's tile pipeline and
//                online softmax over its range;
//   zero_blocks  one per listed empty slot: its output rows set to zero;
//   next_blocks  the next step's staged bookkeeping and KV append.
// The append writes nothing this step's attention reads: the lengths come
// from the kernel arguments, the new token of a sequence of length L goes to
// position L (its last tile's rows past L are zeroed before the value
// product, whatever they hold), its table entries are past the ones read,
// and the host keeps the append in a launch of its own when it would reuse a
// page this step reads (a page freed by a sequence that finished in it).
// An E4M3 append may also re-encode the earlier rows of that page and raise
// its scale; there the unit's own workgroup appends the unit's row once all
// of the unit's reads are done (units_append), and next_blocks only apply
// the bookkeeping.

constexpr int kUnitThreads = kUnitWaves * kWave;

// LDS of an attention workgroup: the waves' K regroup stages (sized for
// bf16 tiles, which E4M3 tiles fit), then every wave's final state,
// lane-major (D / 4 accumulator values, m and l per lane): 100 KB for D = 128,
// which gfx950's 160 KB of LDS per CU holds.
template <int D>
constexpr int unit_state_floats() { return D / 4 + 2; }
template <int D>
constexpr int unit_stage_bytes() { return kUnitWaves * kPageSize * D * 2; }
template <int D>
constexpr int unit_smem_bytes() { return unit_stage_bytes<D>() + kUnitWaves * unit_state_floats<D>() * kWave * 4; }

// Device-scope (cross-XCD coherent) accesses to the piece slots: buffer
// loads and stores with the SC1 cache-policy bit. Unlike atomic accesses
// they are ordinary memory operations for the compiler, so many can be in
// flight at once.
constexpr int kCachePolicyDevice = 16;   // SC1
__device__ __forceinline__ __amdgpu_buffer_rsrc_t piece_rsrc(const float *base, size_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(base), 0, (int)bytes, kRawBufferWord3);
}
__device__ __forceinline__ void store4_device(__amdgpu_buffer_rsrc_t r, int off, f32x4_t v)
{
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, v), r, off, 0, kCachePolicyDevice);
}
__device__ __forceinline__ void store2_device(__amdgpu_buffer_rsrc_t r, int off, f32x2_t v)
{
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2_t, v), r, off, 0, kCachePolicyDevice);
}
__device__ __forceinline__ f32x4_t load4_device(__amdgpu_buffer_rsrc_t r, int off)
{
    return __builtin_bit_cast(f32x4_t, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, kCachePolicyDevice));
}
__device__ __forceinline__ f32x2_t load2_device(__amdgpu_buffer_rsrc_t r, int off)
{
    return __builtin_bit_cast(f32x2_t, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, kCachePolicyDevice));
}

// This lane's part of the argument arrays, fetched before anything else so
// that it arrives together with the scalar arguments.
struct UnitArgs {
    int32_t f_lo, f_hi, seq_lo, seq_hi, len_lo, len_hi, split_lo, split_hi;
};
__device__ __forceinline__ UnitArgs unit_args(const UnitStepParams &up, int lane)
{
    return UnitArgs{up.first[lane + 1],   up.first[lane + 1 + kWave], up.seq[lane],   up.seq[lane + kWave],
                    up.len[lane],         up.len[lane + kWave],       (int32_t)up.split[lane], (int32_t)up.split[lane + kWave]};
}

struct UnitFlags {
    int32_t bad[kUnitWaves];   // per wave: an invalid length, or a page outside the pool
    int32_t last;              // this workgroup is its unit's last to arrive
};

template <int D, bool FP8>
__device__ __forceinline__ void unit_attention(const UnitStepParams &up, const UnitArgs &ar, int blk, uint8_t *smem,
                                               UnitFlags *flags)
{
    const SplitParams &p = up.cur;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int lane = threadIdx.x & (kWave - 1);
    const int n = lane & 15, quad = lane >> 4;
    const int G = p.group, Hkv = p.num_kv_heads;

    // Entry e with first[e] <= blk < first[e + 1], head g and piece k: the
    // argument arrays, read by all lanes at once, are searched in registers (a
    // binary search over them is a chain of dependent loads).
    static_assert(kMaxUnitEntries == 2 * kWave, "the argument arrays are read in two halves");
    const int e = __builtin_popcountll(__builtin_amdgcn_ballot_w64(lane < up.n_entries && ar.f_lo <= blk)) +
                  __builtin_popcountll(__builtin_amdgcn_ballot_w64(lane + kWave < up.n_entries && ar.f_hi <= blk));
    auto pick = [](int lo, int hi, int i) {
        return i < kWave ? __builtin_amdgcn_readlane(lo, i & (kWave - 1)) : __builtin_amdgcn_readlane(hi, i & (kWave - 1));
    };
    const int first_e = e > 0 ? pick(ar.f_lo, ar.f_hi, e - 1) : 0;
    const uint32_t split = (uint32_t)pick(ar.split_lo, ar.split_hi, e);
    const int K = (int)(split & 63u) + 1;
    const int local = blk - first_e;
    const int g = small_div(local, K), k = local - g * K;
    const int b = pick(ar.seq_lo, ar.seq_hi, e);
    const int L = pick(ar.len_lo, ar.len_hi, e);
    const int max_len = p.max_blocks * kPageSize;
    const int Lc = min(L, max_len);
    const int nb = pages_of(L, max_len);
    const uint32_t row0 = (uint32_t)(b * p.num_q_heads + g * G);
    const int next_page = FP8 && up.units_append ? up.next_page[e] : -1;   // fetched ahead of the tail that needs it
    if (nb == 0) {   // the host lists sequences of length >= 1 only; defined anyway: zero rows
        if (k == 0)
            for (int i = threadIdx.x; i < G * D / 8; i += kUnitThreads)
                reinterpret_cast<u32x4_t *>(p.out + (size_t)row0 * D)[i] = u32x4_t{0u, 0u, 0u, 0u};
        return;
    }

    // The unit's next-step rows (E4M3), K by the first half of the waves and V
    // by the second: what they need (it is complete since the last launch) is
    // fetched here by every workgroup of the unit, ahead of the stream, and
    // written once all of the unit's reads are done, these included.
    static_assert(kUnitWaves == 8, "four wavefronts each append K and V");
    const bool tail_append = FP8 && up.units_append && append_valid(up.next, L + 1, next_page);
    AppendE4m3<D, 4> app;
    if (tail_append) {
        app.load_row(up.next, b * Hkv + g, wave / 4, lane);
        app.load_tile(up.next, g, wave / 4, next_page, wave % 4, lane);
    }

    // This wave's tiles [t0, t0 + nt) of the unit: the host's quotient and
    // remainder of nb over the waves, the first waves taking one tile more.
    const int per = (int)(split >> 16), rem = (int)(split >> 6 & 1023u), gw = k * kUnitWaves + wave;
    const int t0 = gw * per + min(gw, rem);
    const int nt = per + (gw < rem ? 1 : 0);

    Piece<D> st;
    reset(st);
    bool bad = L > max_len;
    if (nt > 0) {
        uint8_t *lds = smem + wave * (kPageSize * D * 2);
        const int32_t *bt_row = p.block_table + (size_t)b * p.max_blocks + t0;
        const __amdgpu_buffer_rsrc_t ids_rsrc = buffer_of(bt_row, (uint32_t)nt * 4u);
        int32_t ids = (int32_t)__builtin_amdgcn_raw_buffer_load_b32(ids_rsrc, 4 * lane, 0, 0);
        u32x4_t qop[D / 32];
        load_q<D, FP8>(qop, p, row0, true, n, quad);
        // Chunks of up to 64 tiles, whose block-table entries a wave holds in
        // one register; kDepth tiles in flight within a chunk (one to six
        // measured the same or slower, as did two tiles per step: a wave has
        // three tiles or so, and an odd one costs a whole step). The ids are
        // not loaded inside the tile loop: a load on some iterations only
        // would make every iteration wait for all tiles in flight.
        constexpr int kDepth = kPipelineDepth;
        for (int c0 = 0; c0 < nt; c0 += kWave) {
            const int cn = min(kWave, nt - c0);
            if (c0 > 0)
                ids = (int32_t)__builtin_amdgcn_raw_buffer_load_b32(ids_rsrc, 4 * (c0 + lane), 0, 0);
            // Per lane: issue_step's tile index of tile c0 + lane of the range.
            const bool in = (uint32_t)ids < (uint32_t)p.num_pages;
            const int32_t tile = in ? ids * Hkv + g : ~0;
            bad |= __builtin_amdgcn_ballot_w64(!in && lane < cn) != 0;
            auto issue = [&](Tile<D, FP8> (&t)[1], int i) {   // tile c0 + i of the range, if there is one
                const int32_t T = __builtin_amdgcn_readlane(tile, i & (kWave - 1));
                issue_tile<D, FP8, true>(t[0], p, (uint32_t)(T ^ (T >> 31)), i < cn && T >= 0, n, quad, lane);
            };
            Tile<D, FP8> buf[kDepth][1];
            bf16x8_t qb[D / 32];
#pragma unroll
            for (int s = 0; s < D / 32; ++s)
                qb[s] = __builtin_bit_cast(bf16x8_t, qop[s]);
#pragma unroll
            for (int k0 = 0; k0 < kDepth - 1; ++k0)
                issue(buf[k0], k0);
            for (int i0 = 0; i0 < cn; i0 += kDepth) {
#pragma unroll
                for (int kk = 0; kk < kDepth; ++kk) {
                    const int i = i0 + kk;
                    issue(buf[(kk + kDepth - 1) % kDepth], i + kDepth - 1);
                    if (i < cn) {
                        const int live = min(kPageSize, Lc - (t0 + c0 + i) * kPageSize);   // >= 1: t0 + c0 + i < nb
                        compute_step<D, FP8, 1>(st, buf[kk], qb, p.scale_log2, live, lds, lane, n, quad);
                    }
                }
            }
        }
    }

    // Every wave leaves its state in its own LDS area (past the regroup
    // stages, so nothing needs to wait for them), then one barrier: per lane
    // D/16 groups of four columns (group 4 c + r: r D/16 + 4 c + 0..3 of the
    // lane's quarter of a row), then (m, l). Lanes without a query row hold
    // nothing.
    f32x4_t *const state_acc = reinterpret_cast<f32x4_t *>(smem + unit_stage_bytes<D>());   // [wave][D/16][lane]
    f32x2_t *const state_ml = reinterpret_cast<f32x2_t *>(state_acc + kUnitWaves * (D / 16) * kWave);   // [wave][lane]
    {
        const float lsum = quad_sum(st.l);
        if (n < G) {
            f32x4_t *dst = state_acc + wave * (D / 16) * kWave + lane;
#pragma unroll
            for (int c = 0; c < D / 64; ++c)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    dst[(4 * c + r) * kWave] = f32x4_t{st.acc[4 * c][r], st.acc[4 * c + 1][r], st.acc[4 * c + 2][r],
                                                       st.acc[4 * c + 3][r]};
            state_ml[wave * kWave + lane] = f32x2_t{st.m, lsum};
        }
    }
    if (tail_append)
        app.landed();
    // (The library's barrier with a vote costs two barriers more and a load of
    // the launch's hidden arguments.)
    if (lane == 0)
        flags->bad[wave] = bad ? 1 : 0;
    __syncthreads();
    int32_t any = 0;
#pragma unroll
    for (int w = 0; w < kUnitWaves; ++w)
        any |= flags->bad[w];
    const bool bad_any = any != 0;
    const float poison = bad_any ? __builtin_nanf("") : 0.0f;

    // Combine the kUnitWaves states, in wave order (so the result does not
    // depend on timing). An item is one group of four columns of one row;
    // consecutive threads take consecutive rows. (As single floats, 34 stores
    // per lane and 48 loads per item, and with the library's vote and arguments
    // fetched one by one, the mean step of a generation took 0.6 us longer.)
    const int unit = e * Hkv + g;
    const int mls = unit_ml_stride(G);
    const __amdgpu_buffer_rsrc_t ml_rsrc = piece_rsrc(p.part_ml, sizeof(float) * kMaxUnitBlocks * mls);
    const __amdgpu_buffer_rsrc_t acc_rsrc = piece_rsrc(p.part_acc, sizeof(float) * kMaxUnitBlocks * G * D);
    for (int item = threadIdx.x; item < G * (D / 4); item += kUnitThreads) {
        const int w4 = small_div(item, G), cn = item - w4 * G;   // (c, r, quad) of its columns; row
        const int cq = w4 & 3, cr = (w4 >> 2) & 3, c = w4 >> 4;
        const int cl = cn + 16 * cq;                         // source lane
        float m[kUnitWaves], ls[kUnitWaves];
        f32x4_t x[kUnitWaves];
#pragma unroll
        for (int w = 0; w < kUnitWaves; ++w) {
            const f32x2_t ml = state_ml[w * kWave + cl];
            m[w] = ml[0];
            ls[w] = ml[1];
            x[w] = state_acc[(w * (D / 16) + 4 * c + cr) * kWave + cl];
        }
        float M = m[0];
#pragma unroll
        for (int w = 1; w < kUnitWaves; ++w)
            M = fmaxf(M, m[w]);
        float l = 0.0f;
        f32x4_t a = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < kUnitWaves; ++w) {
            const float wt = m[w] == kNegInf ? 0.0f : __builtin_amdgcn_exp2f(m[w] - M);
            l += wt * ls[w];
            a += wt * x[w];
        }
        const int col = cq * (D / 4) + cr * (D / 16) + 4 * c;
        if (K == 1) {   // the whole unit: normalise and write the columns
            const float inv = bad_any ? __builtin_nanf("") : 1.0f / l;
            *reinterpret_cast<u32x2_t *>(p.out + ((size_t)row0 + cn) * D + col) =
                u32x2_t{pack_bf16(a[0] * inv, a[1] * inv), pack_bf16(a[2] * inv, a[3] * inv)};
        } else {
            // A piece goes to slot blk; the last of the unit's K workgroups
            // to arrive merges them. The pieces cross XCDs, whose L2 caches
            // are not coherent with each other, so they are written and read
            // with device-scope accesses (each goes to the coherent level
            // itself), and the writers' stores complete before the count. An
            // agent-scope fence would do the same by writing back, or
            // invalidating, the whole L2 of the XCD, at several microseconds
            // per workgroup.
            store4_device(acc_rsrc, 4 * ((blk * G + cn) * D + col), a + poison);
            if (w4 == 0)
                store2_device(ml_rsrc, 4 * (blk * mls + 2 * cn), f32x2_t{M + poison, l});
        }
    }
    if (K == 1) {
        if (tail_append)   // the only workgroup: its waves have loaded since the barrier above
            app.store(L + 1, wave % 4, lane);
        return;
    }
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_s_waitcnt(0);   // this wave's part of the piece has reached the coherent level
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __syncthreads();
    if (threadIdx.x == 0)
        flags->last = __hip_atomic_fetch_add(up.counters + unit, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == K - 1;
    __syncthreads();
    if (flags->last == 0)
        return;
    // Every workgroup of the unit has counted its arrival after its loads
    // returned, so none reads the unit's pages any more.
    if (tail_append)
        app.store(L + 1, wave % 4, lane);
    // The last arrival merges the unit's K pieces (slots first[e] + g K ..),
    // in slot order, row j and four columns per thread. Up to eight pieces:
    // every load at once; more: the (m, l) pairs through LDS first, then
    // eight pieces' columns at a time.
    const int slot0 = first_e + g * K;
    if (K <= 8) {
        for (int idx = threadIdx.x; idx < G * (D / 4); idx += kUnitThreads) {
            const int j = idx / (D / 4), c = (idx - j * (D / 4)) * 4;
            f32x2_t ml[8];
            f32x4_t a[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                if (u < K) {
                    ml[u] = load2_device(ml_rsrc, 4 * ((slot0 + u) * mls + 2 * j));
                    a[u] = load4_device(acc_rsrc, 4 * (((slot0 + u) * G + j) * D + c));
                }
            }
            float M = kNegInf;
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (u < K)
                    M = fmaxf(M, ml[u][0]);
            float l = 0.0f;
            f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                if (u < K) {
                    const float w = ml[u][0] == kNegInf ? 0.0f : __builtin_amdgcn_exp2f(ml[u][0] - M);
                    l += w * ml[u][1];
                    acc += w * a[u];
                }
            }
            const float inv = 1.0f / l;
            *reinterpret_cast<u32x2_t *>(p.out + ((size_t)row0 + j) * D + c) =
                u32x2_t{pack_bf16(acc[0] * inv, acc[1] * inv), pack_bf16(acc[2] * inv, acc[3] * inv)};
        }
    } else {
        f32x2_t *const s_ml = reinterpret_cast<f32x2_t *>(smem);   // [K][G], in the regroup stages
        for (int q = threadIdx.x; q < K * G; q += kUnitThreads) {
            const int pq = q / G, j = q - pq * G;
            s_ml[q] = load2_device(ml_rsrc, 4 * ((slot0 + pq) * mls + 2 * j));
        }
        __syncthreads();
        for (int idx = threadIdx.x; idx < G * (D / 4); idx += kUnitThreads) {
            const int j = idx / (D / 4), c = (idx - j * (D / 4)) * 4;
            float M = kNegInf;
            for (int q = 0; q < K; ++q)
                M = fmaxf(M, s_ml[q * G + j][0]);
            float l = 0.0f;
            f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
            for (int q0 = 0; q0 < K; q0 += 8) {
                f32x4_t a[8];
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    if (q0 + u < K)
                        a[u] = load4_device(acc_rsrc, 4 * (((slot0 + q0 + u) * G + j) * D + c));
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    if (q0 + u < K) {
                        const f32x2_t ml = s_ml[(q0 + u) * G + j];
                        const float w = ml[0] == kNegInf ? 0.0f : __builtin_amdgcn_exp2f(ml[0] - M);
                        l += w * ml[1];
                        acc += w * a[u];
                    }
                }
            }
            const float inv = 1.0f / l;
            *reinterpret_cast<u32x2_t *>(p.out + ((size_t)row0 + j) * D + c) =
                u32x2_t{pack_bf16(acc[0] * inv, acc[1] * inv), pack_bf16(acc[2] * inv, acc[3] * inv)};
        }
    }
    if (threadIdx.x == 0)   // for the next launch (ordered by the kernel boundary)
        __hip_atomic_store(up.counters + unit, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <int D, bool FP8>
__global__ __launch_bounds__(kUnitThreads) void engine_unit_step_kernel(UnitStepParams up)
{
    __shared__ __attribute__((aligned(16))) uint8_t smem[unit_smem_bytes<D>()];
    __shared__ UnitFlags flags;
    const UnitArgs ar = unit_args(up, threadIdx.x & (kWave - 1));
    // Scalar arguments are loaded where they are first used, and the first touch
    // of each 64-byte line of them is a trip to memory (a launch's arguments are
    // in no cache), several in a row on the way to the first tile. Naming a field
    // of every line has them come with the arrays, in one trip.
    asm volatile("" ::"s"(up.cur.q), "s"(up.cur.batch), "s"(up.cur.num_pages), "s"(up.next.num_pages), "s"(up.n_entries),
                 "s"(up.next_blocks), "v"(ar.f_lo), "v"(ar.f_hi), "v"(ar.seq_lo), "v"(ar.seq_hi), "v"(ar.len_lo),
                 "v"(ar.len_hi), "v"(ar.split_lo), "v"(ar.split_hi));
    int blk = (int)blockIdx.x;
    if (blk < up.unit_blocks) {
        unit_attention<D, FP8>(up, ar, blk, smem, &flags);
        return;
    }
    blk -= up.unit_blocks;
    if (blk < up.zero_blocks) {
        u32x4_t *dst = reinterpret_cast<u32x4_t *>(up.cur.out + (size_t)up.zero[blk] * up.cur.num_q_heads * D);
        for (int i = threadIdx.x; i < up.cur.num_q_heads * D / 8; i += kUnitThreads)
            dst[i] = u32x4_t{0u, 0u, 0u, 0u};
        return;
    }
    blk -= up.zero_blocks;
    apply_stage<kUnitWaves * kWave>(up.next, blk, up.next_blocks);
    if (up.units_append)
        return;
    const int unit = blk * kUnitWaves + (int)(threadIdx.x / kWave);
    if (unit < up.next.batch * up.next.num_kv_heads)
        append_unit_bf16<D>(up.next, unit, threadIdx.x & (kWave - 1));
}

}  // namespace

hipError_t launch_unit_step(const UnitStepParams &up, int head_dim, bool fp8, hipStream_t stream)
{
    const dim3 grid((unsigned)(up.unit_blocks + up.zero_blocks + up.next_blocks)), block(kUnitThreads);
    if (grid.x == 0)
        return hipSuccess;
    if (head_dim == 128 && !fp8)
        hipLaunchKernelGGL((engine_unit_step_kernel<128, false>), grid, block, 0, stream, up);
    else if (head_dim == 64 && !fp8)
        hipLaunchKernelGGL((engine_unit_step_kernel<64, false>), grid, block, 0, stream, up);
    else if (head_dim == 128 && fp8)
        hipLaunchKernelGGL((engine_unit_step_kernel<128, true>), grid, block, 0, stream, up);
    else if (head_dim == 64 && fp8)
        hipLaunchKernelGGL((engine_unit_step_kernel<64, true>), grid, block, 0, stream, up);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_engine_fill(const int32_t *pages, int n_pages, int hkv, int head_dim, bool fp8, uint32_t seed,
                              void *k_pages, void *v_pages, float *k_scales, float *v_scales, hipStream_t stream)
{
    const dim3 grid((unsigned)(n_pages * hkv)), block(kEngineThreads);
    if (head_dim == 128 && !fp8)
        hipLaunchKernelGGL((engine_fill_kernel<128, false>), grid, block, 0, stream, pages, hkv, seed, k_pages,
                           v_pages, k_scales, v_scales);
    else if (head_dim == 64 && !fp8)
        hipLaunchKernelGGL((engine_fill_kernel<64, false>), grid, block, 0, stream, pages, hkv, seed, k_pages,
                           v_pages, k_scales, v_scales);
    else if (head_dim == 128 && fp8)
        hipLaunchKernelGGL((engine_fill_kernel<128, true>), grid, block, 0, stream, pages, hkv, seed, k_pages,
                           v_pages, k_scales, v_scales);
    else if (head_dim == 64 && fp8)
        hipLaunchKernelGGL((engine_fill_kernel<64, true>), grid, block, 0, stream, pages, hkv, seed, k_pages,
                           v_pages, k_scales, v_scales);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace sl
