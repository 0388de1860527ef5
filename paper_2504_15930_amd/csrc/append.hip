// KV append kernel: every workgroup runs append_block (append_unit.h, which
// states the rules); in the engine's staged mode the launch also applies the
// step's lengths and block-table updates.
#include "append_unit.h"

namespace sl {
namespace {

template <int D, int KIND>
__global__ __launch_bounds__(kAppendThreads) void append_kernel(AppendParams p)
{
    const int blk = blockIdx.x;
    // Nothing in this launch reads the lengths or the block table from memory in this mode.
    if (p.stage)
        apply_stage<kAppendThreads>(p, blk, gridDim.x);
    append_block<D, KIND>(p, blk);
}

}  // namespace

hipError_t launch_append(const AppendParams &p, int head_dim, bool fp8, hipStream_t stream)
{
    const AppendKind kind = append_kind(p, fp8);
    // Fewer than 2^24 units, so at most 2^22 workgroups: a dimension holds fewer than 2^32 threads.
    const dim3 grid((unsigned)append_blocks(p, kind)), block(kAppendThreads);
#define SL_APPEND(DD, KK) \
    if (head_dim == DD && kind == KK) \
        hipLaunchKernelGGL((append_kernel<DD, KK>), grid, block, 0, stream, p); \
    else
    SL_APPEND(128, kAppendBf16)
    SL_APPEND(64, kAppendBf16)
    SL_APPEND(128, kAppendSpread)
    SL_APPEND(64, kAppendSpread)
    SL_APPEND(128, kAppendWave)
    SL_APPEND(64, kAppendWave)
        return hipErrorInvalidValue;
#undef SL_APPEND
    return hipGetLastError();
}

}  // namespace sl
