#ifndef SL_WAVE_OPS_H
#define SL_WAVE_OPS_H
// Reductions and scans over the 64 lanes of a wavefront with DPP operand
// moves: a vector instruction per step, where a shuffle is a round trip
// through LDS (some 50 ns, six of them per reduction).
#include <hip/hip_runtime.h>

namespace sl {
namespace {

// The 32-bit value of the lane that the DPP control names, or `none` where
// there is no such lane or its row of 16 is masked out.
template <int CTRL, int ROWS, class T>
__device__ __forceinline__ T lane_from(T x, T none)
{
    static_assert(sizeof(T) == 4, "one register");
    return __builtin_bit_cast(T, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, none), __builtin_bit_cast(int, x),
                                                             CTRL, ROWS, 0xf, false));
}

// Inclusive scan under Op (op(a, b), kIdentity): shifts by 1, 2, 4 and 8
// within rows of 16 lanes, then the row totals passed on.
template <class Op, class T>
__device__ __forceinline__ T wave_scan(T x)
{
    constexpr T kNone = Op::kIdentity;
    x = Op::op(x, lane_from<0x111, 0xf>(x, kNone));
    x = Op::op(x, lane_from<0x112, 0xf>(x, kNone));
    x = Op::op(x, lane_from<0x114, 0xf>(x, kNone));
    x = Op::op(x, lane_from<0x118, 0xf>(x, kNone));
    x = Op::op(x, lane_from<0x142, 0xa>(x, kNone));
    return Op::op(x, lane_from<0x143, 0xc>(x, kNone));
}

// Reductions: the last lane's scan, in every lane.
template <class Op, class T>
__device__ __forceinline__ T wave_reduce(T x)
{
    return __builtin_bit_cast(T, __builtin_amdgcn_readlane(__builtin_bit_cast(int, wave_scan<Op>(x)), 63));
}

struct FloatMax {
    static constexpr float kIdentity = -__builtin_inff();
    __device__ static float op(float a, float b) { return __builtin_fmaxf(a, b); }
};
struct FloatSum {
    static constexpr float kIdentity = 0.0f;
    __device__ static float op(float a, float b) { return a + b; }
};
__device__ __forceinline__ float wave_max(float x) { return wave_reduce<FloatMax>(x); }
__device__ __forceinline__ float wave_sum(float x) { return wave_reduce<FloatSum>(x); }

}  // namespace
}  // namespace sl

#endif  // SL_WAVE_OPS_H
