// wave_ops.h -- wavefront reductions for gfx950 kernels (DPP moves inside rows of
// 16 lanes, readlane across rows); every sum is taken in a fixed order, so equal
// inputs give equal bits.
#pragma once

#include <hip/hip_runtime.h>

#include "amg_internal.h"

namespace amg {
namespace {

// Cross-lane moves inside rows of 16 lanes (DPP, no LDS traffic): exchange with
// lane ^ 1 and lane ^ 2 inside a quad, mirror inside 8 lanes, mirror inside 16.
constexpr int kDppQuadXor1 = 0xB1, kDppQuadXor2 = 0x4E, kDppRowHalfMirror = 0x141, kDppRowMirror = 0x140;
template <int CTRL>
__device__ inline double dpp_f64(double v)
{
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xF, 0xF, false);
    return __hiloint2double(hi, lo);
}
// Sum over each row of 16 lanes, received by every lane of the row: each step adds
// the partner's partial sum, and both partners form the same sum (fixed order).
// The lanes of the row must be active.
__device__ inline double row16_sum(double v)
{
    v += dpp_f64<kDppQuadXor1>(v);
    v += dpp_f64<kDppQuadXor2>(v);
    v += dpp_f64<kDppRowHalfMirror>(v);
    v += dpp_f64<kDppRowMirror>(v);
    return v;
}
// v of one lane, as a wavefront-uniform value
__device__ inline double lane_value(double v, int lane)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                            __builtin_amdgcn_readlane(__double2loint(v), lane));
}
// Sum over the wavefront, the same value in every lane (fixed order).  All lanes
// must be active.
__device__ inline double wave_sum(double v)
{
    v = row16_sum(v);
    return (lane_value(v, 0) + lane_value(v, 16)) + (lane_value(v, 32) + lane_value(v, 48));
}

// Sum over each aligned group of G lanes, received by every lane of the group
// (fixed order).  The moves stay inside the group, so lanes of other groups may
// be inactive.
template <int G>
__device__ inline double group_sum(double v)
{
    if (G >= 2) v += dpp_f64<kDppQuadXor1>(v);
    if (G >= 4) v += dpp_f64<kDppQuadXor2>(v);
    if (G >= 8) v += dpp_f64<kDppRowHalfMirror>(v);
    if (G >= 16) v += dpp_f64<kDppRowMirror>(v);
    if (G >= 32) v += __shfl_xor(v, 16, kWave);
    if (G >= 64) v += __shfl_xor(v, 32, kWave);
    return v;
}

// Cross-lane moves that keep lane % 4: rotations inside rows of 16 lanes, then the
// exchange of rows (gfx950's permlane swaps: with both operands equal they give the
// even and the odd rows, the low and the high half).
constexpr int kDppRowRor4 = 0x124, kDppRowRor8 = 0x128;
__device__ __forceinline__ double rows_pair_sum(double v)  // over two neighbouring rows of 16
{
    const auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(v), __double2loint(v), false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(v), __double2hiint(v), false, false);
    return __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
}
__device__ __forceinline__ double halves_sum(double v)  // over the two halves of the wavefront
{
    const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(v), __double2loint(v), false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(v), __double2hiint(v), false, false);
    return __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
}
// Sum over the lanes with the same lane % 4 (lanes 0 to 3 hold the result)
__device__ __forceinline__ double mod4_sum(double v)
{
    v += dpp_f64<kDppRowRor4>(v);
    v += dpp_f64<kDppRowRor8>(v);
    return halves_sum(rows_pair_sum(v));
}
// Sums of four values over the wavefront: lane d (0 to 3) receives the d-th.  The four
// values are first spread over the lanes (after two exchanges lane t holds one of them,
// summed over its quad), so one chain of moves reduces all four: about a third of the
// instructions of four separate sums.
__device__ __forceinline__ double spread4_sum(const double (&v)[4])
{
    const int lane = threadIdx.x & (kWave - 1);
    const bool b0 = lane & 1, b1 = lane & 2;
    const double x = (b0 ? v[1] : v[0]) + dpp_f64<kDppQuadXor1>(b0 ? v[0] : v[1]);
    const double y = (b0 ? v[3] : v[2]) + dpp_f64<kDppQuadXor1>(b0 ? v[2] : v[3]);
    return mod4_sum((b1 ? y : x) + dpp_f64<kDppQuadXor2>(b1 ? x : y));
}

}  // namespace
}  // namespace amg
