// Group-relative advantage (Eq. 2 of arXiv 2505.18573) of ONE rollout group, computed by
// one wave: A_i = (r_i - mean(r)) / std(r), two passes over the group's rewards (mean,
// then squared deviations), sums in fp64.  A group whose rewards are all identical gets
// exactly 0 (Section 4.2), decided by max == min.  Shared by the stand-alone kernel and by
// the training-side vocabulary pass, which can carry the groups along in the same launch.
//
// Bound by one chain of dependent instructions: offsets, rewards, two reductions, a square root and a division.
// Up to 64 rollouts stay in a register each, and the reductions run on DPP (64 groups of 8 on MI355X: 3.4 us with
// the rewards read three times and reductions through LDS permutes, 2.9 us so).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "vocab_common.h"

namespace e3 {

__device__ __forceinline__ void advantages_of_group(const float* __restrict__ rewards,
                                                    const int32_t* __restrict__ offsets, int g,
                                                    int32_t ddof, float eps, float* __restrict__ adv,
                                                    int lane)
{
    const int64_t lo = offsets[g], hi = offsets[g + 1];
    const int64_t n = hi - lo;
    if (n <= 0) return;

    if (n <= 64) {
        const bool mine = lane < n;
        const float r = rewards[lo + (mine ? lane : 0)];          // the others repeat the first, for the extremes
        if (wave_max(r) == -wave_max(-r)) {
            if (mine) adv[lo + lane] = 0.0f;
            return;
        }
        const double mean = wave_sum(mine ? (double)r : 0.0) / (double)n;
        const double d = mine ? (double)r - mean : 0.0;
        const double denom = sqrt(wave_sum(d * d) / (double)(n - ddof)) + (double)eps;
        if (mine) adv[lo + lane] = (float)(d / denom);
        return;
    }
    double sum = 0.0;
    float rmax = -INFINITY, rmin = INFINITY;
    for (int64_t i = lo + lane; i < hi; i += 64) {
        const float r = rewards[i];
        sum += (double)r;
        rmax = fmaxf(rmax, r);
        rmin = fminf(rmin, r);
    }
    sum = wave_sum(sum);
    rmax = wave_max(rmax);
    rmin = -wave_max(-rmin);
    if (rmax == rmin) {
        for (int64_t i = lo + lane; i < hi; i += 64) adv[i] = 0.0f;
        return;
    }
    const double mean = sum / (double)n;
    double ss = 0.0;
    for (int64_t i = lo + lane; i < hi; i += 64) {
        const double d = (double)rewards[i] - mean;
        ss += d * d;
    }
    const double denom = sqrt(wave_sum(ss) / (double)(n - ddof)) + (double)eps;
    for (int64_t i = lo + lane; i < hi; i += 64)
        adv[i] = (float)(((double)rewards[i] - mean) / denom);
}

}  // namespace e3
