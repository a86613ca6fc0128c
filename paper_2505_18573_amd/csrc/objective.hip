// Forward value of the GRPO clipped objective (Eq. 1 of arXiv 2505.18573, without the
// KL term the paper drops): per token min(r A, clip(r, 1-eps, 1+eps) A) with
// r = exp(logp_new - logp_old), averaged over the tokens of a rollout, then over the
// rollouts of a question, then over questions.  It consumes what the vocabulary pass
// (log-probs) and the advantage kernel (A) produce.  Two launches: one to sixteen waves per
// rollout (fp64 sums, DPP reductions), then one workgroup that folds rollouts into questions
// and questions into the scalar; every sum has an order fixed by the shape (bit-reproducible).
#include "vocab_common.h"
#include "vocab_pass.h"

namespace e3 {

// The terms of one rollout, kWaves waves of a workgroup each.  The kernel moves 12 bytes per
// token and is bound by latency, not by bytes: what counts is how many tokens are requested at
// once, hence several waves per rollout and up to kUnroll tokens per lane requested before the
// first is used - as many as the rollout has left, rounded up to a power of two, so that a short one
// does not request its tokens several times.  512 rollouts of 77 - 8192 tokens (1.6 M tokens,
// 19 MB) on MI355X: one wave per rollout with one token per lane at a time 44.2 us, this form 6.8 us
// (2.8 TB/s).
constexpr int kUnroll = 8;

template <int kWaves, int kSeqsPerBlock>
__global__ __launch_bounds__(kWaves * kSeqsPerBlock * 64)
void grpo_seq_terms_kernel(const float* __restrict__ logp_new, const float* __restrict__ logp_old,
                           const int32_t* __restrict__ seq_offsets, const float* __restrict__ adv,
                           int32_t num_seqs, float clip_eps, float* __restrict__ token_term_out,
                           double* __restrict__ seq_mean_out)
{
    static_assert(kWaves == 1 || kSeqsPerBlock == 1, "waves of several rollouts do not meet at one barrier");
    constexpr int kStep = kWaves * 64;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int i = blockIdx.x * kSeqsPerBlock + (kWaves == 1 ? wave : 0);
    if (i >= num_seqs) return;
    const int64_t t0 = seq_offsets[i], t1 = seq_offsets[i + 1];
    const float A = adv[i];
    const float lo = 1.0f - clip_eps, hi = 1.0f + clip_eps;
    double acc = 0.0;
    // kN steps of the rollout's waves from token t on, requested together.  (Not quite: in blocks of two steps and more the compiler moves the first
    // step's two requests behind the branch on its bound, where they wait once more, after the others have left.)
    auto terms = [&](auto steps, int64_t t) {
        constexpr int kN = decltype(steps)::value;
        float n[kN], o[kN];
#pragma unroll
        for (int u = 0; u < kN; ++u) {
            const int64_t tu = t + u * kStep < t1 ? t + u * kStep : t0;
            n[u] = logp_new[tu];
            o[u] = logp_old[tu];
        }
#pragma unroll
        for (int u = 0; u < kN; ++u) {
            const float r = __builtin_amdgcn_exp2f((n[u] - o[u]) * kLog2eF);
            const float rc = fminf(fmaxf(r, lo), hi);
            const float term = fminf(r * A, rc * A);
            if (t + u * kStep < t1) {
                if (token_term_out) token_term_out[t + u * kStep] = term;
                acc += (double)term;
            }
        }
    };
    int64_t t = t0 + (kWaves == 1 ? lane : (int)threadIdx.x);
    for (int64_t left = (t1 - t0 + kStep - 1) / kStep; left > 0; left -= kUnroll, t += kStep * kUnroll) {     // uniform
        if (left > 4) terms(std::integral_constant<int, kUnroll>{}, t);
        else if (left > 2) terms(std::integral_constant<int, 4>{}, t);
        else if (left > 1) terms(std::integral_constant<int, 2>{}, t);
        else terms(std::integral_constant<int, 1>{}, t);
    }
    acc = wave_sum(acc);
    if (kWaves > 1) {
        __shared__ double partial[kWaves];
        if (lane == 0) partial[wave] = acc;
        __syncthreads();
        if (threadIdx.x != 0) return;
        acc = 0.0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) acc += partial[w];
    }
    if (lane == 0) seq_mean_out[i] = t1 > t0 ? acc / (double)(t1 - t0) : 0.0;
}

// Questions to the scalar, one workgroup, bound by the latency of its dependent requests (a
// question's two offsets, then its rollouts' means): kLanes lanes share a question while a single round
// of the 1024 threads takes all questions, one lane each beyond that, so that more lanes never
// cost more rounds (a whole call with eight lanes for any number of questions / so: 512 questions x 8
// rollouts of 300 tokens 10.9 / 8.9 us, 20,000 questions of one rollout 124 / 20 us; 64 questions x 8: the
// fold alone 4.5 us with one lane per question, 1.9 us with eight).  A question's sum and the fold over
// questions have an order fixed by the shape.
template <int kLanes>
__global__ __launch_bounds__(1024)
void grpo_objective_reduce_kernel(const double* __restrict__ seq_mean,
                                  const int32_t* __restrict__ group_offsets, int32_t num_groups,
                                  double* __restrict__ objective_out)
{
    static_assert(kLanes == 1 || kLanes == 2 || kLanes == 4 || kLanes == 8, "lanes of one row of sixteen");
    __shared__ double partial[16];
    double acc = 0.0;
    const int sub = threadIdx.x & (kLanes - 1);
    const auto offset = [&](int64_t q) -> int32_t { return group_offsets[q < num_groups ? q : num_groups]; };
    int64_t q = threadIdx.x / kLanes;
    int32_t i0 = 0, i1 = 0;
    if (num_groups > 0) { i0 = offset(q); i1 = offset(q + 1); }
    for (int64_t q0 = 0; q0 < num_groups; q0 += 1024 / kLanes) {   // whole waves take part in the reductions
        q += 1024 / kLanes;
        const int32_t next0 = offset(q), next1 = offset(q + 1);    // requested ahead of these sums
        double g = 0.0;
#pragma unroll 4
        for (int32_t i = i0 + sub; i < i1; i += kLanes) g += seq_mean[i];
        if (kLanes >= 2) g += dpp_d<kDppXor1>(0.0, g);
        if (kLanes >= 4) g += dpp_d<kDppXor2>(0.0, g);
        if (kLanes >= 8) g += dpp_d<kDppHalfMirror>(0.0, g);        // the other four of the eight
        if (sub == 0 && i1 > i0) acc += g / (double)(i1 - i0);
        i0 = next0; i1 = next1;
    }
    acc = wave_sum(acc);
    if ((threadIdx.x & 63) == 0) partial[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        double total = 0.0;
        for (int w = 0; w < 16; ++w) total += partial[w];
        *objective_out = num_groups > 0 ? total / (double)num_groups : 0.0;
    }
}

template <int kWaves, int kSeqsPerBlock>
static void launch_terms(dim3 blocks, const float* logp_new, const float* logp_old, const int32_t* seq_offsets,
                         const float* adv, int32_t num_seqs, float clip_eps, float* token_term_out,
                         double* seq_mean_out, hipStream_t stream)
{
    hipLaunchKernelGGL((grpo_seq_terms_kernel<kWaves, kSeqsPerBlock>), blocks, dim3(kWaves * kSeqsPerBlock * 64), 0,
                       stream, logp_new, logp_old, seq_offsets, adv, num_seqs, clip_eps, token_term_out, seq_mean_out);
}

hipError_t launch_grpo_objective(const float* logp_new, const float* logp_old,
                                 const int32_t* seq_offsets, const float* adv, int32_t num_seqs,
                                 const int32_t* group_offsets, int32_t num_groups, float clip_eps,
                                 float* token_term_out, double* seq_mean_out, double* objective_out,
                                 hipStream_t stream)
{
    if (num_seqs > 0) {
        // The waves per rollout: 16, 8, 4 or 2 while all of them are resident at once (32 per compute
        // unit), else one.  Long and very different rollouts gain from waves, short ones pay for launching
        // idle ones.  512 rollouts of up to 8192 tokens 9.0 us with eight waves, 8.3 with sixteen, of up to 2048 4.9
        // and 5.3; 2048 of up to 8192 27.2 us with one wave, 20.5 with two, 18.0 with four, of 100 tokens
        // 5.8, 6.0 and 6.3; 3072 of up to 4096 17.6, 14.7 and (four, not all resident) 13.6 us; 4096 of 100
        // tokens 6.0, 6.5 and 7.3.
        const int64_t resident = 32 * (int64_t)compute_units();
        const dim3 one((unsigned)num_seqs);
        if (num_seqs * (int64_t)16 <= resident) launch_terms<16, 1>(one, logp_new, logp_old, seq_offsets, adv, num_seqs, clip_eps, token_term_out, seq_mean_out, stream);
        else if (num_seqs * (int64_t)8 <= resident) launch_terms<8, 1>(one, logp_new, logp_old, seq_offsets, adv, num_seqs, clip_eps, token_term_out, seq_mean_out, stream);
        else if (num_seqs * (int64_t)4 <= resident) launch_terms<4, 1>(one, logp_new, logp_old, seq_offsets, adv, num_seqs, clip_eps, token_term_out, seq_mean_out, stream);
        else if (num_seqs * (int64_t)2 <= resident) launch_terms<2, 1>(one, logp_new, logp_old, seq_offsets, adv, num_seqs, clip_eps, token_term_out, seq_mean_out, stream);
        else launch_terms<1, 4>(dim3((unsigned)(((int64_t)num_seqs + 3) / 4)), logp_new, logp_old, seq_offsets, adv, num_seqs, clip_eps, token_term_out, seq_mean_out, stream);
        hipError_t err = hipGetLastError();
        if (err != hipSuccess) return err;
    }
    auto reduce = num_groups <= 1024 / 8 ? grpo_objective_reduce_kernel<8>
                : num_groups <= 1024 / 4 ? grpo_objective_reduce_kernel<4>
                : num_groups <= 1024 / 2 ? grpo_objective_reduce_kernel<2> : grpo_objective_reduce_kernel<1>;
    hipLaunchKernelGGL(reduce, dim3(1), dim3(1024), 0, stream, seq_mean_out, group_offsets, num_groups, objective_out);
    return hipGetLastError();
}

}  // namespace e3
