// KV append kernel: every workgroup runs append_block (append_unit.h, which
// states the rules); in the engine's staged mode the launch also applies the
// step's lengths and block-table updates.
#include "append_unit.h"

namespace sl {
namespace {

template <int D, bool FP8>
__global__ __launch_bounds__(kAppendThreads) void append_kernel(AppendParams p)
{
    const int blk = blockIdx.x;
    // Nothing in this launch reads the lengths or the block table from memory in this mode.
    if (p.stage)
        apply_stage<kAppendThreads>(p, blk, gridDim.x);
    append_block<D, FP8>(p, blk);
}

}  // namespace

hipError_t launch_append(const AppendParams &p, int head_dim, bool fp8, hipStream_t stream)
{
    const long long units = (long long)p.batch * p.num_kv_heads;
    // Fewer than 2^24 units, so at most 2^22 workgroups: a dimension holds fewer than 2^32 threads.
    const dim3 grid((unsigned)(fp8 ? append_blocks<true>(units) : append_blocks<false>(units)));
    const dim3 block(kAppendThreads);
    if (head_dim == 128 && !fp8)
        hipLaunchKernelGGL((append_kernel<128, false>), grid, block, 0, stream, p);
    else if (head_dim == 64 && !fp8)
        hipLaunchKernelGGL((append_kernel<64, false>), grid, block, 0, stream, p);
    else if (head_dim == 128 && fp8)
        hipLaunchKernelGGL((append_kernel<128, true>), grid, block, 0, stream, p);
    else if (head_dim == 64 && fp8)
        hipLaunchKernelGGL((append_kernel<64, true>), grid, block, 0, stream, p);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace sl
