// Prefix sums over the 64 lanes of a wave on DPP, shared by the two restricted samplers: four shifts inside each row of
// sixteen lanes, then lane 15 of a row into the next row and lane 31 into the upper half (lanes that a shift does
// not reach read zero).  All lanes of the wave take part.
#pragma once
#include "vocab_common.h"

namespace e3 {

// Inclusive prefix sums.
__device__ __forceinline__ int wave_prefix_sum(int v)
{
    v += __builtin_amdgcn_mov_dpp(v, 0x111, 0xF, 0xF, true);      // row_shr:1
    v += __builtin_amdgcn_mov_dpp(v, 0x112, 0xF, 0xF, true);      // row_shr:2
    v += __builtin_amdgcn_mov_dpp(v, 0x114, 0xF, 0xF, true);      // row_shr:4
    v += __builtin_amdgcn_mov_dpp(v, 0x118, 0xF, 0xF, true);      // row_shr:8
    v += dpp_i<kDppBcast15, 0xA>(0, v);
    v += dpp_i<kDppBcast31, 0xC>(0, v);
    return v;
}
__device__ __forceinline__ double wave_prefix_sum(double v)
{
    v += dpp_all<0x111>(v);
    v += dpp_all<0x112>(v);
    v += dpp_all<0x114>(v);
    v += dpp_all<0x118>(v);
    v += dpp_d<kDppBcast15, 0xA>(0.0, v);
    v += dpp_d<kDppBcast31, 0xC>(0.0, v);
    return v;
}

// A count and a mass together, so that neither waits for its own additions.
__device__ __forceinline__ void wave_prefix_sum2(int c, double m, int& C, double& M)
{
    auto shift = [&](auto by) {
        constexpr int kCtrl = decltype(by)::value;
        const int x = __builtin_amdgcn_mov_dpp(c, kCtrl, 0xF, 0xF, true);
        const double y = dpp_all<kCtrl>(m);
        c += x; m += y;
    };
    shift(std::integral_constant<int, 0x111>{}); shift(std::integral_constant<int, 0x112>{});
    shift(std::integral_constant<int, 0x114>{}); shift(std::integral_constant<int, 0x118>{});
    { const int x = dpp_i<kDppBcast15, 0xA>(0, c); const double y = dpp_d<kDppBcast15, 0xA>(0.0, m); c += x; m += y; }
    { const int x = dpp_i<kDppBcast31, 0xC>(0, c); const double y = dpp_d<kDppBcast31, 0xC>(0.0, m); c += x; m += y; }
    C = c; M = m;
}
// The same inside each row of sixteen lanes.
__device__ __forceinline__ void row16_prefix_sum2(int c, double m, int& C, double& M)
{
    auto shift = [&](auto by) {
        constexpr int kCtrl = decltype(by)::value;
        const int x = __builtin_amdgcn_mov_dpp(c, kCtrl, 0xF, 0xF, true);
        const double y = dpp_all<kCtrl>(m);
        c += x; m += y;
    };
    shift(std::integral_constant<int, 0x111>{}); shift(std::integral_constant<int, 0x112>{});
    shift(std::integral_constant<int, 0x114>{}); shift(std::integral_constant<int, 0x118>{});
    C = c; M = m;
}

}  // namespace e3
