// Prefix sums over the 64 lanes of a wave on DPP, shared by the two restricted samplers: four shifts inside each row of
// sixteen lanes, then lane 15 of a row into the next row and lane 31 into the upper half (lanes that a shift does
// not reach read zero).  All lanes of the wave take part.
#pragma once
#include "vocab_common.h"

namespace e3 {

// Inclusive prefix sums.
__device__ __forceinline__ int wave_prefix_sum(int v)
{
    v += dpp_i<0x111>(0, v);               // row_shr:1
    v += dpp_i<0x112>(0, v);               // row_shr:2
    v += dpp_i<0x114>(0, v);               // row_shr:4
    v += dpp_i<0x118>(0, v);               // row_shr:8
    v += dpp_i<kDppBcast15, 0xA>(0, v);
    v += dpp_i<kDppBcast31, 0xC>(0, v);
    return v;
}
__device__ __forceinline__ double wave_prefix_sum(double v)
{
    v += dpp_d<0x111>(0.0, v);
    v += dpp_d<0x112>(0.0, v);
    v += dpp_d<0x114>(0.0, v);
    v += dpp_d<0x118>(0.0, v);
    v += dpp_d<kDppBcast15, 0xA>(0.0, v);
    v += dpp_d<kDppBcast31, 0xC>(0.0, v);
    return v;
}

}  // namespace e3
