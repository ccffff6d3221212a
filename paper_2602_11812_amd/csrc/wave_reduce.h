// Wave-wide (64 lanes) reductions by a fixed xor tree: every lane ends up with the result, and the
// order of the additions is the same in every run.  Device-side header.
//
// The exchanges stay in the vector unit: inside a row of 16 lanes by data-parallel-primitive moves (once the lanes of a
// quad agree, mirroring eight lanes pairs each quad with its neighbour, and so on), across rows by swapping rows or halves
// of two registers.  Through the LDS crossbar, as __shfl_xor goes, each of the six steps is an LDS latency
// (head_layer1_skinny_kernel, 63 exchanges: 8.0 -> 7.1 us at d = 4096, d_h = 1024, 4.6 instead of 5.6 at small sizes).
#pragma once
#include <hip/hip_runtime.h>

namespace egtp {
namespace {

// op over lane pairs at distances 1, 2, 4, 8, 16, 32
template <class Op>
__device__ __forceinline__ float wave_tree(float v, Op op)
{
    constexpr int XOR1 = 0xB1, XOR2 = 0x4E, HALF_MIRROR = 0x141, MIRROR = 0x140;  // quad_perm, quad_perm, within 8, within 16
#define EGTP_DPP(ctrl) \
    __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(v), ctrl, 0xf, 0xf, true))
    v = op(v, EGTP_DPP(XOR1));
    v = op(v, EGTP_DPP(XOR2));
    v = op(v, EGTP_DPP(HALF_MIRROR));
    v = op(v, EGTP_DPP(MIRROR));
#undef EGTP_DPP
    const auto rows = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = op(__uint_as_float(rows[0]), __uint_as_float(rows[1]));
    const auto halves = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return op(__uint_as_float(halves[0]), __uint_as_float(halves[1]));
}

__device__ __forceinline__ float wave_sum(float v)
{
    return wave_tree(v, [](float a, float b) { return a + b; });
}

__device__ __forceinline__ float wave_max(float v)
{
    return wave_tree(v, [](float a, float b) { return fmaxf(a, b); });
}

// one halving step on the first n of a[]: lanes whose bit is set keep the upper half of the indices, the others the lower,
// each adding what its partner `ctrl` (a lane with that bit flipped) passes on
template <int CTRL, int N>
__device__ __forceinline__ void halve_in_row(float (&a)[64], bool upper)
{
#pragma unroll
    for (int i = 0; i < N / 2; ++i) {
        const float keep = upper ? a[i + N / 2] : a[i];
        const float pass = upper ? a[i] : a[i + N / 2];
        a[i] = keep + __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(pass), CTRL, 0xf, 0xf, true));
    }
}

// a[0] of lane l = the sum over all lanes of a[l], by the same means: swapping halves or rows of two registers is the exchange
// and the choice of what to keep in one
__device__ __forceinline__ void halve_over_lanes(float (&a)[64])
{
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int i = 0; i < 32; ++i) {
        const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(a[i]), __float_as_uint(a[i + 32]), false, false);
        a[i] = __uint_as_float(s[0]) + __uint_as_float(s[1]);
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(a[i]), __float_as_uint(a[i + 16]), false, false);
        a[i] = __uint_as_float(s[0]) + __uint_as_float(s[1]);
    }
    constexpr int ROTATE8 = 0x128, HALF_MIRROR = 0x141, XOR2 = 0x4E, XOR1 = 0xB1;
    halve_in_row<ROTATE8, 16>(a, lane & 8);
    halve_in_row<HALF_MIRROR, 8>(a, lane & 4);
    halve_in_row<XOR2, 4>(a, lane & 2);
    halve_in_row<XOR1, 2>(a, lane & 1);
}

}  // namespace
}  // namespace egtp
