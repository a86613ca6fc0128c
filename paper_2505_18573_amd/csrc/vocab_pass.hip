// Vocabulary pass for gfx950: one coalesced HBM read of a [rows, V] logit matrix
// that yields, per row, the entropy of softmax(z / tau), the log-probability of a
// sampled or given token and (rollout side) a two-level Gumbel-max sample.
//
// Paper: arXiv 2505.18573.  Softmax with temperature and the Shannon entropy are
// Appendix A's; the entropy is evaluated through the appendix's decomposition
// H = beta * sum_i p_i Delta_i + ln Z(beta), which in running-reference form is
// H = ln S - W/S with S = sum exp(a_i - ref), W = sum (a_i - ref) exp(a_i - ref).
// The paper samples rollouts "at temperature tau" (Section 5.1) without describing
// a sampler; the two-level Gumbel-max used here is specified in include/e3.h.
//
// Work decomposition (wave = 64 lanes):
//   * a row is cut into super-tiles of 4096 columns; one wave streams a whole
//     super-tile as 8 sweeps of 64 lanes x 8 columns (16 bytes of bf16 per lane),
//     so every load instruction of a wave covers 1 KiB of contiguous memory, and the
//     8 chunks one lane sees are exactly one sampler tile;
//   * a workgroup of 8 waves owns a few whole rows; the super-tiles of those rows are
//     work items dealt to the waves round-robin (wave w takes items w, w + 8, ...), so
//     which columns a wave sums, and in which order, depends on the shape alone and the
//     results are the same bit for bit in every run; a wave keeps the first sweeps of
//     its next item in flight while it finishes the current one;
//   * a wave accumulates the items it gets from one row in registers (fp32 per lane,
//     one integer-valued log2 reference per wave that moves by exact powers of two)
//     and hands over one partial per row; the wave that delivers a row's last item
//     merges the partials in fp64, runs level 2 of the sampler and writes the outputs
//     while the other waves keep streaming.
#include "advantages.h"
#include "vocab_common.h"
#include "vocab_pass.h"
#include <hip/hip_ext.h>
#include <mutex>

namespace e3 {

// What a wave hands over for one row (also: the row's incomplete super-tile).
struct alignas(16) RowPartial {
    double S, W;       // sums over the wave's columns except `top`, relative to rc
    float rc, top;     // reference and excluded maximum; rc = -inf marks an empty slot
    float q;           // mass / E of the best sampler tile among them, relative to rc
    int tile;          // its tile id
};
static_assert(sizeof(RowPartial) == 32, "layout");

// What a wave tells the others about its first work item before the streaming starts: a
// logit value that the item's row holds (see the floor in start_row).
struct WaveHint { int row; float value; };
constexpr int kMaxWaves = 8;

// LDS layout: WaveHint hints[kMaxWaves] | uint32 done[rpb] (padded to 16 B)
//             | RowPartial parts[rpb][kWaves+1] | float inv_e[rpb][nst][64]   (rollout side only)
__host__ __device__ inline size_t lds_done_bytes(int rpb)
{
    return sizeof(WaveHint) * kMaxWaves + (size_t)((rpb * 4 + 15) / 16 * 16);
}

template <int kWaves>
__host__ __device__ inline size_t lds_bytes(int rpb, int nst, bool sample)
{
    return lds_done_bytes(rpb) + sizeof(RowPartial) * (size_t)rpb * (kWaves + 1)
         + (sample ? (size_t)rpb * nst * kLanes * sizeof(float) : 0);
}

// Logits of -1e10, or 1e10, and beyond lie up to 2^-24 of themselves off their fp32 reference (see reference_for), which can make
// the sums of a wave infinite.  As a rule these are masked columns, to be scaled away: to zero, so what is handed over is finite.  A
// row that overflows with its own largest columns is no number, as the value tells.
constexpr double kOverflow = 0x1p200;          // no sum of fp32 terms comes near it
constexpr float kHugeReference = 0x1p31f;      // below it a reference is off by 64 at most, which all sums bear
__device__ __forceinline__ void finite_sums(RowPartial& p)
{
    // (NaN stays; products with a distance between references, up to 2^128, stay finite)
    p.S = p.S > kOverflow ? 0x1p800 : p.S;
    p.W = p.W > kOverflow ? 0x1p800 : p.W;
    p.q = fminf(p.q, 3.402823466e38f);
    p.top = p.top > kAbsent ? p.top : -INFINITY;                       // (see new_maximum)
}

// A partial brought to the reference R >= its own (exact scaling; an empty one counts nothing).  Its excluded maximum joins the
// sums as an ordinary term unless it is the row's.
__device__ __forceinline__ float scaled_mass(const RowPartial& p, float R)
{
    const double d = (double)R - (double)p.rc;                         // integer >= 0
    return p.rc > -INFINITY ? ldexpf(p.q, d > 4000.0 ? -4000 : -(int)d) : -1.0f;
}
__device__ __forceinline__ void scaled_sums(const RowPartial& p, float R, bool is_peak, double cd, double& S, double& W)
{
    S = 0.0; W = 0.0;
    if (p.rc > -INFINITY) {
        const double d = (double)R - (double)p.rc;
        const int sh = d > 4000.0 ? -4000 : -(int)d;
        S = ldexp(p.S, sh);
        W = ldexp(p.W - d * p.S, sh);
        if (!is_peak && p.top > -INFINITY) {                           // a wave may have excluded nothing
            const double tw = (double)p.top * cd - (double)R;
            // 2^tw, tw <= 0: integer and fraction apart (exact), so that no intermediate leaves fp32's range
            const double whole = rint(tw);
            const double ew = ldexp((double)__builtin_amdgcn_exp2f((float)(tw - whole)), whole < -4000.0 ? -4000 : (int)whole);
            S += ew;
            W += tw * ew;
        }
    }
}

// Several partials of one row (at most sixteen, in LDS) as one, by the first lanes of a wave: the sums at the largest
// reference, every excluded maximum but the largest an ordinary term.
__device__ __forceinline__ RowPartial merge_partials(const RowPartial* parts, int nparts, float c, int lane)
{
    RowPartial p;
    p.S = 0.0; p.W = 0.0; p.rc = -INFINITY; p.top = -INFINITY; p.q = -1.0f; p.tile = 0;
    const int slot = lane & 15;                                        // lanes 16..31 hold them once more
    if (slot < nparts) p = parts[slot];
    float R = p.rc, peak = p.top;
    row16_max2(R, peak);
    const bool is_peak = slot == (int)__builtin_ctzll(__ballot(p.top == peak) | (1ull << 63));
    RowPartial m;
    m.rc = R; m.top = peak;
    const Cand best = row16_best(Cand{scaled_mass(p, R), p.tile});
    double S, W;
    scaled_sums(p, R, is_peak, (double)c, S, W);
    m.q = best.q; m.tile = best.idx;
    const double both = row16_sums(lane < 16 ? S : W);
    m.S = read_lane(both, 0);
    m.W = read_lane(both, 16);
    if (!(fabsf(R) < kHugeReference)) finite_sums(m);                  // uniform
    return m;
}

// Row epilogue, run by one wave once all of the row's partials are written: merge the
// partials (one per lane, nparts <= 64), level 2 of the sampler or the target gather,
// outputs.  kFew: the partials sit in the first sixteen lanes (a row-block workgroup hands
// over at most nine), so every reduction over them is four DPP steps inside one row of lanes
// instead of six across the wave; level 2 always works on sixteen lanes.  This wave's work
// is a chain of dependent instructions that nothing overlaps once the row is the last of the
// launch, hence the care to keep it short: maxima and sums two at a time, races as a maximum and a look at who
// holds it, the winning tile's columns requested without a branch (which made the wave wait for each of them), the
// logarithm and the reciprocal in a few fp64 instructions of their own (vocab_common.h).  4600 cycles for a wave
// with its data in reach before; whole calls, before and now in us: 1 row x 32,000 bf16 6.9 / 6.0, 300 x 1000 7.4 / 6.4,
// 512 x 151,936 28.8 / 27.9, 4096 x 32,000 63.3 / 55.8 (where the vector ALUs are the limit).
template <typename Chunk, bool kSample, bool kFew>
__device__ __forceinline__ void finish_row(const VocabPassArgs& a, int64_t row,
                                           const RowPartial* parts, int nparts, int lane)
{
    const int64_t V = a.V;
    const char* rowp = static_cast<const char*>(a.logits)
                     + row * a.row_stride * (int64_t)Chunk::kElemBytes;
    RowPartial p;
    p.S = 0.0; p.W = 0.0; p.rc = -INFINITY; p.top = -INFINITY; p.q = -1.0f; p.tile = 0;
    // (kFew: the second sixteen lanes hold the same partials once more)
    const int slot = kFew ? lane & 15 : lane;
    if (slot < nparts) p = parts[slot];
    // training side: ask for the target's logit early, use it last
    int64_t tgt = -1;
    float z_tgt = 0.0f;
    if (!kSample) {
        if (a.target_ids != nullptr) tgt = a.target_ids[row];
        const int64_t safe = tgt < 0 ? 0 : (tgt >= V ? V - 1 : tgt);
        z_tgt = Chunk::load_one(rowp, safe);
    }
    const float tau = a.tau_rows ? a.tau_rows[row] : a.tau_scalar;
    const float c = kLog2eF / tau;

    // R is the common reference, `peak` the largest logit of the row; the partial
    // that holds it is the lowest lane with that top, every other excluded maximum
    // joins the rest as an ordinary term.
    float R = p.rc, peak = p.top;
    if (kFew) row16_max2(R, peak);
    else wave_max2(R, peak);
    const unsigned long long holders = __ballot(p.top == peak);
    const int peak_lane = (int)__builtin_ctzll(holders | (1ull << 63));
    const bool is_peak = slot == peak_lane;
    const double cd = (double)c;

    // Rollout side, level 1 across partials first (weights brought to the common
    // reference by exact scaling), so that the columns of the winning tile are
    // requested before the fp64 merge below and arrive while it runs.
    typename Chunk::Four four = {};
    float inv_e2[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    uint32_t w[4] = {0u, 0u, 0u, 0u};
    int64_t col0 = 0;
    bool in_tile = false;
    if (kSample) {
        const Cand mine{scaled_mass(p, R), p.tile};
        const Cand win = kFew ? row16_best(mine) : wave_best(mine);
        const int wst = win.idx / kLanes, wslot = win.idx % kLanes;
        // 2 * kDepth lanes x 4 consecutive columns cover the tile
        col0 = (int64_t)wst * kSuperCols + (int64_t)(lane >> 1) * kSweepCols
             + (int64_t)wslot * kChunk + (lane & 1) * 4;
        // without a branch around it, where the compiler would wait for it; lanes without a column read the row's first
        in_tile = lane < 2 * kDepth && col0 < V;
        four = Chunk::load_four(rowp, in_tile ? col0 : 0);
        const uint64_t grow = a.row_base + (uint64_t)row;
        philox4x32_10((uint32_t)(col0 >> 2), (uint32_t)grow, (uint32_t)(grow >> 32), 2u,
                      (uint32_t)a.seed, (uint32_t)(a.seed >> 32), w);
#pragma unroll
        for (int j = 0; j < 4; ++j) inv_e2[j] = inv_exp_variate(w[j]);   // while the columns arrive
    }

    // Row sums in fp64.
    double S_l, W_l;
    scaled_sums(p, R, is_peak, cd, S_l, W_l);
    double S_rest = S_l, W_rest = W_l;
    if (kFew) {
        // lanes 0..15 add up S, lanes 16..31 W
        const double both = row16_sums(lane < 16 ? S_l : W_l);
        S_rest = read_lane(both, 0);
        W_rest = read_lane(both, 16);
    } else {
        wave_sum2(S_rest, W_rest);
    }
    // With e_p = 2^{t_p} the peak's term, x = S_rest / e_p and y = W_rest / e_p:
    //   ln S = t_p ln2 + log1p(x),   H = ln S - ln2 W / S = log1p(x) + ln2 (t_p x - y) / (1 + x),
    // every piece of which is O(x) when the row is peaked.  t_p lies in (-1, 0] (while the reference is exact, see reference_for).
    const double t_p = (double)peak * cd - (double)R;
    const double inv_ep = (double)__builtin_amdgcn_exp2f((float)-t_p);
    // (a sum that overflowed with the row's own columns is no number: finite_sums)
    const double x = S_rest < kOverflow ? S_rest * inv_ep : __builtin_nan(""), y = W_rest * inv_ep;
    const double l1p = log1p_of(x);
    const double H = fma(kLn2 * (t_p * x - y), reciprocal(1.0 + x), l1p);

    if (lane == 0) {
        if (a.entropy_out) a.entropy_out[row] = (float)H;
        if (a.gap_out) {
            // Appendix A's Delta measured on this row: the probability-weighted mean of
            // z_peak - z_i over all other tokens = tau ln2 (t_p - W_rest / S_rest)
            a.gap_out[row] = S_rest > 0.0 ? (float)((double)tau * kLn2 * (t_p - W_rest / S_rest))
                                          : __builtin_nanf("");
        }
    }
    if (kSample) {
        // Level 2: Gumbel-max inside the winning tile, in race form: maximise
        // 2^{(z - z_peak) c} / E_col.  The row's peak serves as the reference: the winning
        // tile's largest column lies within 2^-34 of it (a tile further down cannot make up
        // the difference with its noise, whose range is 2^-24 .. 17), far from underflow.
        float cz[4], q[4];
        Chunk::unpack_four(four, cz);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const bool ok = in_tile && col0 + j < V;
            q[j] = ok ? __builtin_amdgcn_exp2f((cz[j] - peak) * c) * inv_e2[j] : -1.0f;
        }
        // the lane's best (of equals the lowest column), then the wave's: columns rise with the lane
        const float q01 = fmaxf(q[0], q[1]), q23 = fmaxf(q[2], q[3]);
        const float q_lane = fmaxf(q01, q23);
        const int j_lane = q01 >= q23 ? (q[0] >= q[1] ? 0 : 1) : (q[2] >= q[3] ? 2 : 3);
        const Cand cb = row16_best(Cand{q_lane, q_lane >= 0.0f ? (int)col0 + j_lane : 0x7FFFFFFF});
        int64_t tok = cb.idx;
        if (tok < 0 || tok >= V) tok = 0;                 // only reachable with non-finite input
        if (lane == 0) a.token_out[row] = (int32_t)tok;
        // the lane that holds the token's column writes its log-probability:
        //   ln p = (a_tok - a_peak) - log1p(x)
        if (a.logp_out) {
            const bool holder = lane < 2 * kDepth && cb.idx >= col0 && cb.idx < col0 + 4;
            if (holder) {
                const int j = (int)(cb.idx - col0);
                const float z_tok = j == 0 ? cz[0] : j == 1 ? cz[1] : j == 2 ? cz[2] : cz[3];
                a.logp_out[row] = (float)(((double)z_tok - (double)peak) * cd * kLn2 - l1p);
            }
            // no column won the race (non-finite logits): the row's outputs are NaN
            if (__ballot(holder) == 0 && lane == 0) a.logp_out[row] = __builtin_nanf("");
        }
    } else if (lane == 0 && a.logp_out) {
        float lp = __builtin_nanf("");
        if (tgt >= 0 && tgt < V)
            lp = (float)(((double)z_tgt - (double)peak) * cd * kLn2 - l1p);
        a.logp_out[row] = lp;
    }
}

// Empty state for a row.  `floor` is a logit value known to be below (or -inf: nothing known
// about) the row's maximum: logits up to the floor are ordinary terms of the sums even when
// they exceed everything this wave has met, and only a logit above it becomes the wave's
// excluded maximum.  The row's largest logit lies above every floor, so the wave that meets it
// excludes it, which is all the row merge needs (it keeps the one dominant term of a peaked
// row out of the fp32 sums); what the floor saves is the reference moves for the many running
// maxima a wave would otherwise meet on its way.
__device__ __forceinline__ void start_row(LaneState& s, float floor, float c)
{
    s.top = -INFINITY; s.dom_lane = 0; s.dom_open = false;
    s.thr = floor;
    s.rc = floor > -INFINITY ? reference_for(floor, c) : -INFINITY;
    s.S = s.W = s.sT0 = s.sT1 = s.wT0 = s.wT1 = 0.0f;
    s.best = Cand{-1.0f, 0};
}

// A row's incomplete last super-tile: sweeps in two halves, the guarded loads of a
// half all issued before the first is used; columns past V count as absent.  Returns
// whether this lane's tile holds any column.
template <typename Chunk>
__device__ __forceinline__ bool stream_ragged(LaneState& s, const char* rowp, int64_t cbase,
                                              int64_t lane_col, int64_t V, float c, int lane)
{
    bool any_valid = false;
#pragma unroll 1
    for (int half = 0; half < 2; ++half) {
        const int64_t hbase = cbase + (int64_t)half * (kDepth / 2) * kSweepCols;
        if (hbase - lane_col >= V) break;            // uniform: nothing left
        Chunk rb[kDepth / 2];
#pragma unroll
        for (int i = 0; i < kDepth / 2; ++i)
            if (hbase + i * kSweepCols + kChunk <= V) rb[i].load(rowp, hbase + i * kSweepCols);
#pragma unroll
        for (int i = 0; i < kDepth / 2; ++i) {
            const int64_t col = hbase + i * kSweepCols;
            float z[8];
            bool valid = false;
            if (col + kChunk <= V) {
                rb[i].unpack(z);
                valid = true;
            } else {
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    z[j] = kAbsent;
                    if (col + j < V) { z[j] = Chunk::load_one(rowp, col + j); valid = true; }
                }
            }
            any_valid |= valid;
            if (__any(valid)) accumulate_chunk(s, z, c, lane);
        }
    }
    return any_valid;
}

// (Five waves per SIMD for bf16 and four for fp32: without the bound the row epilogue takes the registers of one of them,
// fp32 134 and three waves: 512 x 40,000 21.0 us instead of 19.1; bf16 4096 x 40,000 74.1 and 70.4.)
template <typename Chunk, bool kSample, int kWaves, int kAhead>
__global__ __launch_bounds__(kWaves * 64, Chunk::kElemBytes == 2 ? 5 : 4)
void vocab_pass_kernel(VocabPassArgs a, int rpb)
{
    static_assert(kAhead >= 1 && kAhead <= kDepth && kDepth % kAhead == 0, "the register ring must close over a super-tile");
    static_assert(kWaves <= kMaxWaves, "one hint slot per wave");
    extern __shared__ __align__(16) char smem[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t V = a.V;
    const int nst = (int)((V + kSuperCols - 1) / kSuperCols);   // super-tiles in a row
    const int nfull = (int)(V / kSuperCols);                    // of which complete
    const int64_t row0 = (int64_t)blockIdx.x * rpb;             // first row of this workgroup
    const int nrows = (int)((a.rows - row0) < rpb ? (a.rows - row0) : rpb);
    // items: the rows' incomplete super-tiles first, then complete ones row by row
    const int n_ragged = nst > nfull ? nrows : 0;
    const int total = n_ragged + nrows * nfull;

    WaveHint* hints = reinterpret_cast<WaveHint*>(smem);
    uint32_t* done = reinterpret_cast<uint32_t*>(smem + sizeof(WaveHint) * kMaxWaves);
    RowPartial* parts = reinterpret_cast<RowPartial*>(smem + lds_done_bytes(rpb));
    float* inv_e_tab = reinterpret_cast<float*>(smem + lds_done_bytes(rpb)
                                                + sizeof(RowPartial) * (size_t)rpb * (kWaves + 1));

    const int64_t row_bytes = a.row_stride * (int64_t)Chunk::kElemBytes;
    const int64_t lane_col = (int64_t)lane * kChunk;            // own columns (incomplete sweeps)
    const int64_t sweep_lane_col = Chunk::sweep_col(lane);      // complete sweeps: see the loaders
    const int tlane = Chunk::tile_lane(lane);                   // tile lane held after unpack_sweep
    const char* base = static_cast<const char*>(a.logits) + row0 * row_bytes;

    // item -> (local row, super-tile)
    auto decode = [&](int item, int& r, int& st) {
        if (item < n_ragged) { r = item; st = nfull; }
        else { const int idx = item - n_ragged; r = idx / nfull; st = idx - r * nfull; }
    };

    // Wave w takes items w, w + kWaves, ...; if the first is a complete super-tile its
    // first sweeps are requested before anything else happens.
    int item = wave;
    bool have = item < total;
    Chunk buf[kAhead];
    int r_cur = 0, st_cur = 0;
    if (have && item >= n_ragged) {
        decode(item, r_cur, st_cur);
        const char* rp = base + r_cur * row_bytes;
        const int64_t b0 = (int64_t)st_cur * kSuperCols + sweep_lane_col;
#pragma unroll
        for (int i = 0; i < kAhead; ++i) buf[i].load_sweep(rp, b0 + i * kSweepCols);
    }

    // Workgroup prologue: empty hand-over slots, and (rollout side) the level-1 noise of all
    // tiles of the workgroup's rows, one Philox block per thread per four tiles.
    for (int i = threadIdx.x; i < rpb; i += kWaves * 64) done[i] = 0;
    for (int i = threadIdx.x; i < rpb * (kWaves + 1); i += kWaves * 64) {
        RowPartial e;
        e.S = 0.0; e.W = 0.0; e.rc = -INFINITY; e.top = -INFINITY; e.q = -1.0f; e.tile = 0;
        parts[i] = e;
    }
    if (kSample) {
        const uint32_t seed_lo = (uint32_t)a.seed, seed_hi = (uint32_t)(a.seed >> 32);
        const int calls = nrows * nst * (kLanes / 4);
        for (int cidx = threadIdx.x; cidx < calls; cidx += kWaves * 64) {
            const int r = cidx / (nst * 16), rem = cidx - r * (nst * 16);   // rem = tile / 4 in the row
            const uint64_t grow = a.row_base + (uint64_t)(row0 + r);
            uint32_t w[4];
            philox4x32_10((uint32_t)rem, (uint32_t)grow, (uint32_t)(grow >> 32), 1u, seed_lo, seed_hi, w);
            float4 v;
            v.x = inv_exp_variate(w[0]); v.y = inv_exp_variate(w[1]);
            v.z = inv_exp_variate(w[2]); v.w = inv_exp_variate(w[3]);
            reinterpret_cast<float4*>(inv_e_tab)[(size_t)r * nst * 16 + rem] = v;
        }
    }
    // Every wave whose first item is a complete super-tile tells the workgroup one logit value
    // that item's row holds: the largest among the sweeps it has requested (they have arrived
    // by now on the rollout side, behind the noise table).  The largest of these per row is
    // the floor the waves start that row with; it depends on the data and the launch shape only.
    {
        float mine = -INFINITY;
        int mine_row = -1;
        if (have && item >= n_ragged) {
#pragma unroll
            for (int i = 0; i < kAhead; ++i) mine = fmaxf(mine, buf[i].some_max());
            mine = wave_max(mine);
            mine_row = r_cur;
        }
        if (lane == 0) hints[wave] = WaveHint{mine_row, mine};
    }
    // Workgroup barrier that orders LDS only: __syncthreads() would also wait for the
    // global loads already in flight (its fence covers global memory) and drain the
    // pipeline for a full memory latency.
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    // floor of local row r: just below the largest hint given for it (-inf: none)
    auto row_floor = [&](int r) -> float {
        float v = -INFINITY;
        if (lane < kWaves) {
            const WaveHint h = hints[lane];
            if (h.row == r) v = h.value;
        }
        v = row16_max(v);
        return v > -INFINITY ? v - fmaxf(fabsf(v) * 0x1p-12f, 1.0e-30f) : -INFINITY;
    };

    // Training side, optional: rollout groups riding along.  The last wave has the fewest
    // items (or as many as the others), so it takes workgroup b's group b before it starts
    // on its own; the loads of its first item are already in flight.  The host asks for
    // this only when there are at most as many groups as workgroups.
    if (!kSample && a.adv_groups > 0 && wave == kWaves - 1 && (int)blockIdx.x < a.adv_groups)
        advantages_of_group(a.adv_rewards, a.adv_offsets, (int)blockIdx.x, a.adv_ddof, a.adv_eps,
                            a.adv_out, lane);

    // Hand over what this wave holds for local row r (n_items of its items); the wave
    // that brings the row's count to nst finishes the row.
    auto deliver = [&](LaneState& s, int r, int slot, int n_items) {
        double Sw = (double)s.S, Ww = (double)s.W;
        wave_sum2(Sw, Ww);
        const Cand wb = kSample ? wave_best(s.best) : Cand{-1.0f, 0};
        uint32_t before = 0;
        if (lane == 0) {
            RowPartial p;
            p.S = Sw; p.W = Ww; p.rc = s.rc; p.top = s.top; p.q = wb.q; p.tile = wb.idx;
            if (!(fabsf(s.rc) < kHugeReference)) finite_sums(p);
            parts[r * (kWaves + 1) + slot] = p;
            // Release: the partial is visible to the workgroup before the counter moves.
            // The fence is restricted to the LDS address space, so it waits for this
            // wave's LDS operations only and leaves its global loads in flight.
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
            before = __hip_atomic_fetch_add(&done[r], (uint32_t)n_items, __ATOMIC_RELAXED,
                                            __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        before = __builtin_amdgcn_readfirstlane(before);
        if ((int)before + n_items == nst) {
            // Acquire: the counter said every other wave's partial of this row is written;
            // order the reads of those partials behind it (LDS only, as above).
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
            finish_row<Chunk, kSample, true>(a, row0 + r, parts + r * (kWaves + 1), kWaves + 1, lane);
        }
    };
    auto row_scale = [&](int r) -> float {
        const float tau = a.tau_rows ? a.tau_rows[row0 + r] : a.tau_scalar;
        return kLog2eF / tau;
    };

    // Incomplete super-tiles come first in the item order, so a wave meets them before it
    // enters the pipelined loop.
    while (have && item < n_ragged) {
        const int next = item + kWaves;
        const int r = item, st = nfull;
        const char* rowp = base + r * row_bytes;
        const float c = row_scale(r);
        const float inv_e = kSample ? inv_e_tab[((size_t)r * nst + st) * kLanes + lane] : 0.0f;
        LaneState s;
        start_row(s, row_floor(r), c);
        const bool any_valid = stream_ragged<Chunk>(s, rowp, (int64_t)st * kSuperCols + lane_col,
                                                    lane_col, V, c, lane);
        close_tile<kSample>(s, st * kLanes + lane, inv_e, any_valid, c, lane);
        deliver(s, r, kWaves, 1);
        item = next;
        have = item < total;
        if (have && item >= n_ragged) {
            decode(item, r_cur, st_cur);
            const char* rp = base + r_cur * row_bytes;
            const int64_t b0 = (int64_t)st_cur * kSuperCols + sweep_lane_col;
#pragma unroll
            for (int i = 0; i < kAhead; ++i) buf[i].load_sweep(rp, b0 + i * kSweepCols);
        }
    }

    if (have) {
        // Pipelined loop over complete super-tiles.  Invariant at the top: (r_cur, st_cur)
        // is a complete super-tile whose first kAhead sweeps are requested into buf.
        // Items come in increasing order, so the rows a wave sees never go back: it
        // accumulates one row in `s` and hands it over when the row changes.
        LaneState s;
        int held = 0;                                    // items of r_cur accumulated in s
        float c = row_scale(r_cur);
        start_row(s, row_floor(r_cur), c);
        const char* rowp = base + r_cur * row_bytes;
        while (true) {
            const int next = item + kWaves;
            const float inv_e = kSample ? inv_e_tab[((size_t)r_cur * nst + st_cur) * kLanes + tlane] : 0.0f;
            const int64_t this_base = (int64_t)st_cur * kSuperCols + sweep_lane_col;
#pragma unroll
            for (int i = 0; i < kDepth - kAhead; ++i) {
                float z[8];
                buf[i % kAhead].unpack_sweep(z, lane);
                buf[i % kAhead].load_sweep(rowp, this_base + (i + kAhead) * kSweepCols);
                accumulate_chunk(s, z, c, lane);
            }
            const bool more = next < total;
            int r_next = r_cur, st_next = 0;
            const char* nrowp = rowp;
            int64_t next_base = 0;
            if (more) {
                decode(next, r_next, st_next);
                nrowp = base + r_next * row_bytes;
                next_base = (int64_t)st_next * kSuperCols + sweep_lane_col;
            }
            // two copies of the last sweeps, with and without the requests for the next item:
            // a request under a condition inside one copy makes the compiler wait for more
            // of the loads in flight than the copy with requests needs to
            if (more) {
#pragma unroll
                for (int i = kDepth - kAhead; i < kDepth; ++i) {
                    float z[8];
                    buf[i % kAhead].unpack_sweep(z, lane);
                    buf[i % kAhead].load_sweep(nrowp, next_base + (i + kAhead - kDepth) * kSweepCols);
                    accumulate_chunk(s, z, c, lane);
                }
            } else {
#pragma unroll
                for (int i = kDepth - kAhead; i < kDepth; ++i) {
                    float z[8];
                    buf[i % kAhead].unpack_sweep(z, lane);
                    accumulate_chunk(s, z, c, lane);
                }
            }
            close_tile<kSample>(s, st_cur * kLanes + tlane, inv_e, true, c, lane);
            ++held;
            if (!more || r_next != r_cur) {
                deliver(s, r_cur, wave, held);
                held = 0;
            }
            if (!more) break;
            if (r_next != r_cur) {
                c = row_scale(r_next);
                rowp = base + r_next * row_bytes;
                start_row(s, row_floor(r_next), c);
            }
            r_cur = r_next;
            st_cur = st_next;
            item = next;
        }
    }
}

// ---------------------------------------------------------------------------
// Small batches.  When the rows are too few to give every compute unit a workgroup
// of whole rows, a row is cut into `nslots` runs of consecutive super-tiles and
// every run gets a workgroup of its own, so that all of the chip's memory
// channels are busy even for a single row; it writes one RowPartial to the workspace, and a second launch
// of one wave per row merges a row's partials exactly as the row-block kernel's
// epilogue does.
//
// Such a launch is bound by latency: the first data arrive after 1 to 2 us, and a wave alone on its SIMD issues an
// instruction every five cycles.  So a super-tile is dealt to kParts waves: a wave takes 64 / kParts of its tiles, several lanes
// share a tile, each reading 16-byte vectors of its own (a wave's request covers whole runs of the row), all vectors are
// requested at once and the level-1 noise is drawn while they are in flight.  With everything in registers the wave's
// maximum comes first and the exponentials need no running reference.  The waves' partials meet in LDS.
// Four waves for every super-tile of fp32 and for a few hundred bf16 ones,
// one wave for more of those, where four times the fixed work per wave would keep the vector ALUs busy longer (see split_plan).
// Against one wave per super-tile with a running reference, both launches, us: bf16 x 151,936, 1 row 7.3 -> 5.7, 4 rows
// 7.6 -> 6.2, 64 rows 10.5 -> 9.0, 128 rows 14.6 -> 12.3; fp32 x 70,005, 100 rows 11.0 -> 10.3, 128 rows 12.6 -> 11.6.
// ---------------------------------------------------------------------------
constexpr int kMaxRun = 4;           // super-tiles of a run: a row has at most 64 runs

template <typename Chunk, int kParts>
struct SplitShape {
    static constexpr int kTiles = kLanes / kParts;                  // tiles of a wave
    static constexpr int kRowVecs = kTiles * Chunk::kHalves;        // vectors of one sweep that belong to them
    static constexpr int kGroups = 64 / kRowVecs;                   // lanes / kRowVecs: which sweeps a lane reads
    static constexpr int kVecs = kDepth / kGroups;                  // vectors of a lane, kGroups sweeps apart
    static_assert(kRowVecs <= 64 && kGroups * kRowVecs == 64 && kGroups <= 4 && kVecs * kGroups == kDepth, "whole shares");
    // lanes that between them hold every tile of the wave once (sharers agree on its mass)
    static constexpr unsigned long long kOnce = (kRowVecs == 64 ? ~0ull : (1ull << (kRowVecs & 63)) - 1ull)
                                              & (Chunk::kHalves == 2 ? 0x5555555555555555ull : ~0ull);
    // a lane's value and those of its tile's other lanes, added up
    static __device__ __forceinline__ float sum(float v)
    {
        if (Chunk::kHalves == 2) v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), kDppXor1, 0xF, 0xF, true));
        if (kGroups >= 2) {
            const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
            v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
        }
        if (kGroups >= 4) {
            const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
            v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
        }
        return v;
    }
};

// One super-tile's share of a wave in two steps: the requests, and what it amounts to (wave-uniform).
template <typename Chunk, int kParts>
struct SplitShare : SplitShape<Chunk, kParts> {
    using Shape = SplitShape<Chunk, kParts>;
    static constexpr int kCols = Chunk::kVecCols;
    u32x4 x[Shape::kVecs];

    static __device__ __forceinline__ int tile_of(int lane, int part)  // in the super-tile
    {
        return part * Shape::kTiles + lane % Shape::kRowVecs / Chunk::kHalves;
    }
    static __device__ __forceinline__ int col_of(int lane, int part)   // of the lane's first vector, in the super-tile
    {
        return tile_of(lane, part) * kChunk + lane % Chunk::kHalves * kCols + lane / Shape::kRowVecs * kSweepCols;
    }
    // Requests without branches.  The 16 bytes that hold a column of the row lie inside its pitch; a vector past
    // the row's end is replaced by its first.
    __device__ __forceinline__ void request(const char* rowp, int st, int nfull, int64_t V, int lane, int part)
    {
        const int64_t col0 = (int64_t)st * kSuperCols + col_of(lane, part);
#pragma unroll
        for (int i = 0; i < Shape::kVecs; ++i) {
            const int64_t col = col0 + i * Shape::kGroups * kSweepCols;
            const int64_t at = st < nfull || col < V ? col : 0;
            x[i] = stream_load(reinterpret_cast<const u32x4*>(rowp + at * Chunk::kElemBytes));
        }
    }
    template <bool kSample>
    __device__ __forceinline__ RowPartial reduce(int st, int nfull, int64_t V, float c, float inv_e, int lane, int part) const
    {
        RowPartial p;
        p.S = 0.0; p.W = 0.0; p.rc = -INFINITY; p.top = -INFINITY; p.q = -1.0f; p.tile = 0;
        // (the lowest column of a wave is the first of its first tile)
        const int64_t first_col = (int64_t)st * kSuperCols;
        if (first_col + part * Shape::kTiles * kChunk >= V) return p;  // uniform
        float z[Shape::kVecs][kCols], cm[Shape::kVecs], most = kAbsent;
#pragma unroll
        for (int i = 0; i < Shape::kVecs; ++i) {
            Chunk::unpack_vec(x[i], z[i]);
            if (st >= nfull) {                                         // columns past V are absent
                const int64_t left = V - (first_col + col_of(lane, part) + i * Shape::kGroups * kSweepCols);
#pragma unroll
                for (int j = 0; j < kCols; ++j) z[i][j] = j < left ? z[i][j] : kAbsent;
            }
            cm[i] = kCols == 8 ? fmax3(fmax3(z[i][0], z[i][1], z[i][2]), fmax3(z[i][3], z[i][kCols - 4], z[i][kCols - 3]),
                                       fmaxf(z[i][kCols - 2], z[i][kCols - 1]))
                               : fmax3(fmax3(z[i][0], z[i][1], z[i][2]), z[i][3], z[i][3]);
            most = fmaxf(most, cm[i]);
        }
        // The wave's maximum is kept out of the sums (see LaneState): all logits that equal it are struck, and
        // those beyond the first come back as ordinary terms.
        const float top = wave_max(most);
        const float rc = uniform_f(reference_for(top, c));
        int struck = 0;
#pragma unroll
        for (int i = 0; i < Shape::kVecs; ++i) {
            if (__any(cm[i] == top)) {
#pragma unroll
                for (int j = 0; j < kCols; ++j) {
                    const bool hit = z[i][j] == top;
                    z[i][j] = hit ? kAbsent : z[i][j];
                    struck += hit;
                }
            }
        }
        float s0 = 0.0f, s1 = 0.0f, w0 = 0.0f, w1 = 0.0f;
#pragma unroll
        for (int i = 0; i < Shape::kVecs; ++i) {
#pragma unroll
            for (int j = 0; j < kCols; ++j) {
                const float t = fmaf(z[i][j], c, -rc);
                const float e = __builtin_amdgcn_exp2f(t);
                if (j & 1) { s1 += e; w1 = fmaf(t, e, w1); }
                else       { s0 += e; w0 = fmaf(t, e, w0); }
            }
        }
        float s = s0 + s1, w = w0 + w1;
        const float t_top = fmaf(top, c, -rc), e_top = __builtin_amdgcn_exp2f(t_top);  // (infinite: see finite_sums)
        const unsigned long long holders = __ballot(struck != 0);
        const float mass = struck != 0 ? fmaf((float)struck, e_top, s) : s;
        if (__any(struck > 1) || (holders & (holders - 1ull)) != 0ull) {               // rare
            const int others = struck - (lane == (int)__builtin_ctzll(holders | 1ull << 63));
            const float again = others > 0 ? (float)others * e_top : 0.0f;
            s += again;
            w = fmaf(t_top, again, w);
        }
        p.S = (double)s; p.W = (double)w;
        wave_sum2(p.S, p.W);
        p.rc = rc; p.top = top;
        if (kSample) {
            const int tile = tile_of(lane, part);
            const bool nonempty = first_col + tile * kChunk < V;
            const Cand mine{nonempty ? Shape::sum(mass) * inv_e : -1.0f, st * kLanes + tile};
            const Cand best = holder_of(mine, Shape::kRowVecs == 16 ? row16_max(mine.q) : wave_max(mine.q), Shape::kOnce);
            p.q = best.q; p.tile = best.idx;
        }
        if (!(fabsf(rc) < kHugeReference)) finite_sums(p);             // uniform
        return p;
    }
};

// 1 / E of level 1 for a sampler tile.
__device__ __forceinline__ float tile_noise(const VocabPassArgs& a, uint64_t grow, int tile)
{
    uint32_t w[4];
    philox4x32_10((uint32_t)(tile >> 2), (uint32_t)grow, (uint32_t)(grow >> 32), 1u,
                  (uint32_t)a.seed, (uint32_t)(a.seed >> 32), w);
    const int k = tile & 3;
    return inv_exp_variate(k == 0 ? w[0] : k == 1 ? w[1] : k == 2 ? w[2] : w[3]);
}

template <typename Chunk, bool kSample, int kParts>
__global__ __launch_bounds__(64 * kParts)
void vocab_split_kernel(VocabPassArgs a, RowPartial* __restrict__ ws, int nslots)
{
    using Share = SplitShare<Chunk, kParts>;
    __shared__ RowPartial parts[kMaxRun * kParts];
    const int lane = threadIdx.x & 63;
    const int part = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t V = a.V;
    const int nst = (int)((V + kSuperCols - 1) / kSuperCols);
    const int nfull = (int)(V / kSuperCols);
    const int64_t row = (int64_t)(blockIdx.x / (unsigned)nslots);
    const int slot = (int)(blockIdx.x - (unsigned)row * (unsigned)nslots);
    const int st_begin = slot * nst / nslots;        // runs differ by at most one super-tile
    const int st_end = (slot + 1) * nst / nslots;
    const char* rowp = static_cast<const char*>(a.logits) + row * a.row_stride * (int64_t)Chunk::kElemBytes;
    const uint64_t grow = a.row_base + (uint64_t)row;

    float c = 0.0f;
    for (int st = st_begin; st < st_end; ++st) {
        Share share;
        share.request(rowp, st, nfull, V, lane, part);
        if (st == st_begin) c = kLog2eF / (a.tau_rows ? a.tau_rows[row] : a.tau_scalar);
        const float inv_e = kSample ? tile_noise(a, grow, st * kLanes + Share::tile_of(lane, part)) : 0.0f;
        const RowPartial p = share.template reduce<kSample>(st, nfull, V, c, inv_e, lane, part);
        if (lane == 0) {
            if (kParts == 1 && st_end - st_begin == 1) ws[(size_t)blockIdx.x] = p;
            else parts[(st - st_begin) * kParts + part] = p;
        }
    }
    if (kParts == 1 && st_end - st_begin == 1) return;
    __syncthreads();
    if (part == 0) {
        const RowPartial m = merge_partials(parts, (st_end - st_begin) * kParts, c, lane);
        if (lane == 0) ws[(size_t)blockIdx.x] = m;
    }
}

// ---------------------------------------------------------------------------
// Narrow rows (at most kNarrowTiles super-tiles, and some wider ones: narrow_serves): a workgroup has a row, and a wave kItems shares (SplitShare) of its super-tiles.
// The whole row is requested at once, the waves meet at one barrier, and the first merges the partials and finishes
// the row: one launch, no running reference, no noise table, nothing that waits for another wave before the barrier.
// Bound by latency up to some hundred rows, then by HBM and the launch of workgroups.  Against the streaming kernel, us: bf16 1 row x
// 1000 5.5 -> 3.6, 64 x 8000 7.4 -> 4.4, 64 x 32,000 7.8 -> 5.9, 512 x 32,000 11.3 -> 9.6, 4096 x 16,000 33.5 -> 25.0 (5.2 TB/s),
// 4096 x 32,000 56.5 -> 51.8; fp32 64 x 16,000 7.6 -> 5.3, 1024 x 32,000 26.7 -> 24.4, 4096 x 8000 30.6 -> 24.3.  (Four rows
// of one super-tile to a workgroup, a wave each: 4096 x 1000 9.6 either way.)
// ---------------------------------------------------------------------------
constexpr int kNarrowTiles = 8;
constexpr int kNarrowWaves = 16;     // of a workgroup at most

template <typename Chunk, bool kSample, int kParts, int kItems>
__global__ __launch_bounds__(64 * kNarrowWaves)
void vocab_narrow_kernel(VocabPassArgs a)
{
    using Share = SplitShare<Chunk, kParts>;
    __shared__ RowPartial parts[kNarrowWaves];                         // of sixteen shares at most: one row of lanes merges them
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int waves = (int)(blockDim.x >> 6);
    const int64_t V = a.V;
    const int nfull = (int)(V / kSuperCols);
    const int64_t row = blockIdx.x;
    const char* rowp = static_cast<const char*>(a.logits) + row * a.row_stride * (int64_t)Chunk::kElemBytes;
    const uint64_t grow = a.row_base + (uint64_t)row;

    // item i: part i % kParts of super-tile i / kParts; wave w has the items w and, of two, w + waves
    Share share[kItems];
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
        const int item = wave + i * waves;
        share[i].request(rowp, item / kParts, nfull, V, lane, item % kParts);
    }
    const float c = kLog2eF / (a.tau_rows ? a.tau_rows[row] : a.tau_scalar);
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
        const int item = wave + i * waves, st = item / kParts, part = item % kParts;
        const float inv_e = kSample ? tile_noise(a, grow, st * kLanes + Share::tile_of(lane, part)) : 0.0f;
        const RowPartial p = share[i].template reduce<kSample>(st, nfull, V, c, inv_e, lane, part);
        if (lane == 0) parts[item] = p;
    }
    __syncthreads();
    if (wave == 0) finish_row<Chunk, kSample, true>(a, row, parts, waves * kItems, lane);
    // Training side, optional: workgroup b computes group b's advantages (see vocab_pass_kernel), here beside the row's last
    // steps.  (While the columns are on their way it held 36 registers beside theirs: fp32 1000 x 20,000 25.1 us, 20.7 so.)
    if (!kSample && a.adv_groups > 0 && wave == waves - 1 && (int)blockIdx.x < a.adv_groups)
        advantages_of_group(a.adv_rewards, a.adv_offsets, (int)blockIdx.x, a.adv_ddof, a.adv_eps, a.adv_out, lane);
}

template <typename Chunk, bool kSample>
__global__ __launch_bounds__(64)
void row_finish_kernel(VocabPassArgs a, const RowPartial* __restrict__ ws, int nslots)
{
    finish_row<Chunk, kSample, false>(a, (int64_t)blockIdx.x, ws + (size_t)blockIdx.x * nslots, nslots,
                                      (int)threadIdx.x);
}

// ---------------------------------------------------------------------------
// Batch sums for the scheduler's H_t (mean entropy of the current step, Eq. 4) and the mean gap:
// one workgroup, fp64, fixed summation order (thread t takes rows t, t + 1024, ...).  Bound by
// latency: a thread's next eight rows are requested together (32,768 masked entropies: one row at a time behind its mask
// 21.0 us, so 7.2 us), and entropies and gaps share a launch (1000 rows: two launches 4 us each, one 3.9 us).  With a mask the
// compiler waits for the first row's byte before the other requests leave and reads its value in the branch behind it:
// three waits for eight rows, one without a mask.
// ---------------------------------------------------------------------------
template <bool kGap, bool kMask>
__global__ __launch_bounds__(1024)
void entropy_reduce_kernel(const float* __restrict__ entropy, const float* __restrict__ gap,
                           const uint8_t* __restrict__ mask, int64_t rows, double* sum_out,
                           double* gap_sum_out, int64_t* count_out)
{
    constexpr int kAhead = 8;
    __shared__ double ssum[16], sgap[16], scnt[16];
    double acc = 0.0, acc_gap = 0.0, cnt = 0.0;                   // the count is exact in fp64
    for (int64_t r0 = threadIdx.x; r0 < rows; r0 += 1024 * kAhead) {
        float h[kAhead], g[kAhead];
        uint8_t keep[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const int64_t r = r0 + 1024 * u < rows ? r0 + 1024 * u : r0;     // no branch between the requests
            h[u] = entropy[r];
            if (kGap) g[u] = gap[r];
            keep[u] = kMask ? mask[r] : (uint8_t)1;
        }
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            if (keep[u] && r0 + 1024 * u < rows) {
                acc += (double)h[u];
                if (kGap) acc_gap += (double)g[u];
                cnt += 1.0;
            }
        }
    }
    acc = wave_sum(acc);
    if (kGap) acc_gap = wave_sum(acc_gap);
    cnt = wave_sum(cnt);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) { ssum[wave] = acc; sgap[wave] = acc_gap; scnt[wave] = cnt; }
    __syncthreads();
    if (wave != 0) return;
    const double t = row16_sum(ssum[lane & 15]), tg = kGap ? row16_sum(sgap[lane & 15]) : 0.0, n = row16_sum(scnt[lane & 15]);
    if (lane == 0) {
        if (sum_out) *sum_out = t;
        if (kGap) *gap_sum_out = tg;
        if (count_out) *count_out = (int64_t)n;
    }
}

// ---------------------------------------------------------------------------
// host-side launchers
// ---------------------------------------------------------------------------
constexpr size_t kLdsBudget = 64 * 1024;

// Optional events for the next vocabulary-pass launch of this host thread: `start` gets
// the time the (first) kernel begins to execute, `stop` the time the (last) kernel ends,
// taken from the dispatch itself rather than from marker packets around it.
static thread_local hipEvent_t g_start_event = nullptr;
static thread_local hipEvent_t g_stop_event = nullptr;

void set_launch_events(hipEvent_t start, hipEvent_t stop)
{
    g_start_event = start;
    g_stop_event = stop;
}

LaunchEvents take_launch_events()
{
    LaunchEvents e{g_start_event, g_stop_event};
    g_start_event = nullptr;
    g_stop_event = nullptr;
    return e;
}

// Rows per workgroup of a large batch: at least two items per wave (one row of 38 super-tiles
// at V = 151,936 gives a wave 4 or 5), and the noise table must fit LDS
// (0 = does not fit).  launch_for takes fewer where the batch is too small for that.  Two 8-wave workgroups are resident per compute unit; what exceeds
// that is handed out by the hardware dispatcher as workgroups finish.
template <int kWaves>
static int rows_per_group(int64_t V, bool sample)
{
    const int nst = (int)((V + kSuperCols - 1) / kSuperCols);
    int rpb = (2 * kWaves + nst - 1) / nst;
    if (rpb < 1) rpb = 1;
    while (rpb > 1 && lds_bytes<kWaves>(rpb, nst, sample) > kLdsBudget) --rpb;
    if (lds_bytes<kWaves>(rpb, nst, sample) > kLdsBudget) return 0;
    return rpb;
}

bool vocab_pass_fits(int64_t V) { return rows_per_group<8>(V, true) > 0 && rows_per_group<4>(V, true) > 0; }

int compute_units()
{
    static int cus = 0;
    if (cus == 0) {
        int dev = 0;
        hipDeviceProp_t prop;
        if (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&prop, dev) == hipSuccess)
            cus = prop.multiProcessorCount;
        if (cus <= 0) cus = 256;
    }
    return cus;
}

template <typename Chunk, bool kSample, int kWaves>
static hipError_t launch_groups(const VocabPassArgs& a, int rpb, hipStream_t stream)
{
    if (rpb == 0) return hipErrorInvalidValue;
    const int nst = (int)((a.V + kSuperCols - 1) / kSuperCols);
    const size_t lds = lds_bytes<kWaves>(rpb, nst, kSample);
    const unsigned blocks = (unsigned)((a.rows + rpb - 1) / rpb);
    const LaunchEvents ev = take_launch_events();
    if (ev.start != nullptr || ev.stop != nullptr)
        hipExtLaunchKernelGGL((vocab_pass_kernel<Chunk, kSample, kWaves, Chunk::kAhead>),
                              dim3(blocks), dim3(kWaves * 64), (uint32_t)lds, stream, ev.start, ev.stop, 0u,
                              a, rpb);
    else
        hipLaunchKernelGGL((vocab_pass_kernel<Chunk, kSample, kWaves, Chunk::kAhead>),
                           dim3(blocks), dim3(kWaves * 64), lds, stream, a, rpb);
    return hipGetLastError();
}

// How a batch of whole rows is launched through the streaming kernel.
// Eight waves per workgroup while the whole batch is at most eight workgroups per
// compute unit; four waves per workgroup beyond that, where the hardware dispatcher
// balances across many small groups (measured crossover on MI355X: between 2048 and
// 4096 rows of 151,936 bf16 columns).  Two 8-wave workgroups are resident per compute
// unit: a batch that fills its last round of 2 * CUs workgroups to less than 80 %
// (768 rows on 256 CUs: 512 + 256) runs as 4-wave workgroups if those are all resident
// at once (measured at 768 rows: 45.0 us instead of 49.3 us).
static LaunchPlan streaming_plan(int64_t rows, int64_t V, bool sample)
{
    const int64_t cus = compute_units();
    auto plan = [&](int waves, int rpb) -> LaunchPlan {
        return LaunchPlan{0, 0, waves, rpb, rpb > 0 ? (rows + rpb - 1) / rpb : 0};
    };
    // Several rows per workgroup only where that leaves a resident round of workgroups (nearly) full:
    // 512 rows x 48,000 bf16 columns (two rows per workgroup before) 18.7 -> 15.7 us.
    auto spread = [&](int rpb, int64_t round) -> int {
        const int64_t most = (rows + round / 4) / round;
        return rpb > 1 && most < rpb ? (most > 1 ? (int)most : 1) : rpb;
    };
    const int rpb8 = spread(rows_per_group<8>(V, sample), 2 * cus);
    const int rpb4 = spread(rows_per_group<4>(V, sample), 4 * cus);
    const LaunchPlan eight = plan(8, rpb8), four = plan(4, rpb4);
    if (rpb8 == 0 || eight.workgroups > 8 * cus) return four;
    const int64_t round8 = 2 * cus;
    const int64_t rounds = (eight.workgroups + round8 - 1) / round8;
    if (eight.workgroups > round8 && eight.workgroups * 5 < rounds * round8 * 4 && rpb4 > 0 && four.workgroups <= 4 * cus)
        return four;
    return eight;
}

// Narrow rows: shares per super-tile and per wave; every share has a place in the kernel's table (sixteen).
// While the waves of a batch leave the chip idle, more of them per super-tile are faster; beyond that they only multiply what every
// wave does once.  bf16, one / two / four waves per super-tile, us: 256 rows x 4096 4.7 / 4.4 / 4.2, 512 rows 5.1 / 5.2 / 4.8, 768
// rows 5.3 / 5.3 / 5.5; 256 x 8000 5.3 / 4.8 / 4.8, 512 rows 6.3 / 5.8 / 6.0, 768 rows 6.6 / 6.7 / 6.9; 256 x 16,000 5.7 / 5.6
// / 5.7, 512 rows 7.4 / 7.2 / 7.7, 1024 rows 9.8 / 10.0 / 12.8; 256 x 32,000 7.1 / 6.9, 512 rows 9.9 / 10.1, 2048 rows 29.7 / 29.8.
// fp32 has two to four; more than four super-tiles of two waves each are ten to sixteen waves, of which a compute unit has
// few workgroups at a time, so that larger batches give a wave two shares (us with one / two): 512 x 20,000 10.4 / 11.6, 768 rows
// 15.2 / 13.5; 256 x 32,000 9.0 / 9.5, 512 rows 15.5 / 14.4, 1024 rows 28.2 / 24.5, 4096 rows 95.2 / 80.2.
static LaunchPlan narrow_plan(int64_t rows, int nst, bool is_bf16)
{
    const int64_t cus = compute_units();
    auto plan = [&](int parts, int items) { return LaunchPlan{parts, items, nst * parts / items, 1, rows}; };
    if (!is_bf16) {
        if (nst > 4) return plan(2, rows <= (nst <= 6 ? 2 * cus : cus) ? 1 : 2);
        return plan(rows <= 2 * cus ? 4 : 2, 1);
    }
    if (nst <= 2 && rows * nst <= 2 * cus) return plan(4, 1);
    if (nst > kNarrowTiles) return plan(1, 1);
    return plan(rows <= (nst <= 6 ? 2 * cus : cus) ? 2 : 1, 1);
}

// Which narrow rows have a workgroup each (us, the streaming kernel / so).  Two things speak against it: shares of which a wave has two (86
// registers, training side 110), and a last super-tile with few columns, whose absent ones are worked through, which the streaming
// kernel does not do.
// All bf16 rows but those of eight super-tiles in batches of more than sixteen per compute unit (sampling 3500 x 30,000 39.0 /
// 38.6, 5000 rows 52.3 / 62.4, 10,000 rows 106 / 125; training only with few columns in the last: 10,000 x 28,680 104 / 112, x 32,000 equal).
// fp32 rows of at most four super-tiles, and of more while a wave has one share.  Beyond that
//   - training rows of five or six are streamed (1000 x 17,000 18.4 / 22.0, x 20,000 20.7 / 22.2, x 24,000 22.5 / 24.3);
//   - others up to four (of seven or eight: three and a quarter) per compute unit, where at most half of the last super-tile is
//     filled or all of it (sampling 600 x 20,484 13.1 / 15.1, x 22,000 14.2 / 15.9, x 24,576 14.4 / 15.6, x 26,000 15.6 / 16.0; but x 24,000
//     16.2 / 16.2, x 28,000 18.0 / 16.9, and 1280 x 22,000 26.4 / 24.2), or up to one and a half per compute unit;
//   - and large batches with few columns in the last (training 10,000 x 24,580 152 / 161, sampling 5000 x 28,680 88.5 / 92.0;
//     training rows of seven also from five to eight per compute unit: 2048 x 26,000 36.9 / 40.1, 2400 rows 47.5 / 44.9).
// Rows of nine to sixteen super-tiles, where they are not cut: bf16 with at most a row per compute unit, a wave per super-tile
// (129 x 33,000 9.0 / 6.8, 256 x 50,000 10.3 / 9.1, 256 x 65,000 12.4 / 10.1, 400 x 50,000 12.7 / 14.4).
// A launch has fewer than 2^32 threads: rows of 64 to 256 threads each reach that at 2^24 to 2^26 rows, eight of them to a workgroup of the
// streaming kernel at 2^27.
static bool narrow_serves(int64_t rows, int64_t V, bool is_bf16, bool sample)
{
    const int64_t cus = compute_units();
    const int nst = (int)((V + kSuperCols - 1) / kSuperCols);
    if (nst > kNarrowTiles) return is_bf16 && nst <= kNarrowWaves && rows <= cus;
    if (rows * narrow_plan(rows, nst, is_bf16).waves * 64 > (int64_t)UINT32_MAX) return false;
    const int64_t last = V % kSuperCols;                               // columns of an incomplete last super-tile
    const bool light = last <= kSuperCols / 2, few = light && last != 0;
    if (is_bf16) return nst < 8 || rows <= 16 * cus || !(sample || few);
    if (nst < 5 || rows <= (nst <= 6 ? 2 * cus : cus)) return true;
    if (!sample && nst <= 6) return false;
    if (4 * rows <= (nst <= 6 ? 16 : 13) * cus) return !light && 2 * rows > 3 * cus;
    if (!few || nst == 5) return true;
    if (nst == 6) return rows <= 24 * cus;
    if (nst == 7) return sample || rows <= 5 * cus || (rows > 8 * cus && rows <= 16 * cus);
    return rows <= 16 * cus;
}

// Short rows in large batches: a workgroup of one or two waves, most lanes of which have no column, costs more to launch than to
// run.  Four rows to a workgroup of the streaming kernel, a wave each (us, so / narrow): bf16 training side 5000 x 64 7.7 / 9.4, 8192 x
// 64 11.2 / 13.1, 5000 x 1000 8.7 / 10.0, but 6000 x 750 12.0 / 11.1; fp32 8192 x 500 16.4 / 20.5 and 13.0 / 15.7, training side 5000 x 900 12.3 / 11.2;
// bf16 samples and fp32 rows of at most 256 columns stay narrow (fp32 10,000 x 256 1.0 to 1.05 times as long so).
static bool four_short_rows(int64_t rows, int64_t V, bool is_bf16, bool sample)
{
    const int64_t cus = compute_units();
    if (rows <= 10 * cus || (rows + 3) * 64 > (int64_t)UINT32_MAX) return false;
    if (is_bf16) return !sample && V <= (rows <= 20 * cus ? 1024 : 448);
    return V > 256 && V <= (sample ? 1024 : 768);
}

template <typename Chunk, bool kSample>
static hipError_t launch_narrow(const VocabPassArgs& a, const LaunchPlan& plan, hipStream_t stream)
{
    if (plan.waves * plan.items > kNarrowWaves) return hipErrorInvalidValue;
    auto kernel = plan.parts == 4 ? vocab_narrow_kernel<Chunk, kSample, 4, 1> : vocab_narrow_kernel<Chunk, kSample, 2, 1>;
    if constexpr (Chunk::kHalves == 1) {
        if (plan.parts == 1) kernel = vocab_narrow_kernel<Chunk, kSample, 1, 1>;
    } else {
        if (plan.items == 2) kernel = vocab_narrow_kernel<Chunk, kSample, 2, 2>;
    }
    const LaunchEvents ev = take_launch_events();
    const dim3 blocks((unsigned)plan.workgroups), threads(64u * (unsigned)plan.waves);
    if (ev.start != nullptr || ev.stop != nullptr)
        hipExtLaunchKernelGGL(kernel, blocks, threads, 0u, stream, ev.start, ev.stop, 0u, a);
    else
        hipLaunchKernelGGL(kernel, blocks, threads, 0, stream, a);
    return hipGetLastError();
}

template <typename Chunk, bool kSample>
static hipError_t launch_for(const VocabPassArgs& a, const LaunchPlan& plan, hipStream_t stream)
{
    if (plan.parts != 0) return launch_narrow<Chunk, kSample>(a, plan, stream);
    return plan.waves == 8 ? launch_groups<Chunk, kSample, 8>(a, plan.rows_per_group, stream)
                           : launch_groups<Chunk, kSample, 4>(a, plan.rows_per_group, stream);
}

// Split path: used when the row-block path would leave compute units without a
// workgroup and the caller brought enough workspace.  Every super-tile gets a workgroup of
// its own (measured on MI355X: small workgroups beyond what is resident are handed
// out by the hardware dispatcher as earlier ones finish, which balances better than
// longer static runs), except that a row has at most 64 runs: one partial per lane
// of the merging wave.
// Rows of at most kNarrowTiles super-tiles are not cut: a workgroup holds all of them and needs no second launch (64 rows x
// 32,000 bf16: 5.9 us).  Wider rows are cut while whole rows would make at most half as many workgroups as there are compute
// units.  The line was drawn with kernels that both have since become faster, one wave per super-tile in the one and the streaming
// kernel in the other, and has not been drawn again: for bf16 rows of nine to sixteen super-tiles, narrow when whole, it is
// too high (64 x 33,000 cut 7.4, 129 x 33,000 whole 6.8); rows x 151,936 cut are now 9.0 at 64 and 12.3 at 128.  Then, cut / whole in us, bf16
// samples: 64 rows x 33,000 9.6 / 9.9, x 70,005 10.6 / 13.9, x 151,936 12.1 / 15.1; 128 rows 10.5 / 10.7,
// 12.3 / 14.5, 15.9 / 15.8; 192 rows 11.3 / 11.1, 13.8 / 15.1, 19.0 / 16.8; x 61,000 12.6 / 12.4 at 128 rows and
// 13.7 / 12.6 at 192.  (Rows of a whole number of super-tiles are faster whole at any count, 128 x
// 40,960 11.0 / 9.1; x 61,441, one column into the sixteenth, from 112 rows on by 4 %.)
constexpr int64_t kSplitMaxRows = 1024;          // bound used by the workspace size

struct SplitPlan {
    int nslots;      // runs per row, 1 <= nslots <= min(64, super-tiles per row)
    int waves;       // of a run's workgroup
};

static SplitPlan split_plan(int64_t rows, int64_t V, bool is_bf16)
{
    const int nst = (int)((V + kSuperCols - 1) / kSuperCols);
    SplitPlan p;
    p.nslots = nst < 64 ? nst : 64;
    // One / four waves per super-tile, bf16, us: 8 rows x 33,000 (72 super-tiles) 6.8 / 6.2, 4 x 151,936 (152) 6.7 / 6.2, 32 x 33,000
    // (288) 7.1 / 6.8, 32 x 40,960 (320) 6.6 / 6.7, 64 x 33,000 (576) 7.4 / 7.5, 128 x 70,005 (2304) 9.1 / 10.8; fp32 loads
    // twice the bytes for the same arithmetic: four are faster at every count (100 x 70,005 10.9 / 10.3).
    p.waves = is_bf16 && rows * p.nslots * 4 > (int64_t)compute_units() * 5 ? 1 : 4;
    return p;
}

size_t vocab_pass_workspace_bytes(int64_t rows, int64_t V)
{
    if (rows <= 0 || rows > kSplitMaxRows || V <= 0) return 0;
    const int64_t nst = (V + kSuperCols - 1) / kSuperCols;
    return (size_t)rows * (size_t)(nst < 64 ? nst : 64) * sizeof(RowPartial);
}

template <typename Chunk, bool kSample>
static hipError_t launch_split(const VocabPassArgs& a, RowPartial* ws, SplitPlan plan, hipStream_t stream)
{
    const unsigned blocks = (unsigned)(a.rows * plan.nslots);
    const LaunchEvents ev = take_launch_events();
    const RowPartial* parts = ws;
    auto kernel = vocab_split_kernel<Chunk, kSample, 4>;
    if constexpr (Chunk::kHalves == 1) {
        if (plan.waves == 1) kernel = vocab_split_kernel<Chunk, kSample, 1>;
    }
    if (ev.start != nullptr)
        hipExtLaunchKernelGGL(kernel, dim3(blocks), dim3(64 * plan.waves), 0u, stream,
                              ev.start, (hipEvent_t) nullptr, 0u, a, ws, plan.nslots);
    else
        hipLaunchKernelGGL(kernel, dim3(blocks), dim3(64 * plan.waves), 0, stream,
                           a, ws, plan.nslots);
    hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;
    if (ev.stop != nullptr)
        hipExtLaunchKernelGGL((row_finish_kernel<Chunk, kSample>), dim3((unsigned)a.rows), dim3(64), 0u,
                              stream, (hipEvent_t) nullptr, ev.stop, 0u, a, parts, plan.nslots);
    else
        hipLaunchKernelGGL((row_finish_kernel<Chunk, kSample>), dim3((unsigned)a.rows), dim3(64), 0, stream,
                           a, parts, plan.nslots);
    return hipGetLastError();
}

LaunchPlan vocab_pass_plan(int64_t rows, int64_t V, bool is_bf16, bool sample, bool* cut)
{
    const int64_t nst = (V + kSuperCols - 1) / kSuperCols;
    const bool narrow = narrow_serves(rows, V, is_bf16, sample);
    *cut = false;
    if (four_short_rows(rows, V, is_bf16, sample)) return LaunchPlan{0, 0, 4, 4, (rows + 3) / 4};
    if (nst <= kNarrowTiles && narrow) return narrow_plan(rows, (int)nst, is_bf16);
    const LaunchPlan streaming = streaming_plan(rows, V, sample);
    *cut = nst > kNarrowTiles && rows <= kSplitMaxRows && streaming.workgroups > 0
        && streaming.workgroups * E3_SPLIT_BELOW_DEN <= (int64_t)compute_units() * E3_SPLIT_BELOW_NUM;
    return narrow ? narrow_plan(rows, (int)nst, is_bf16) : streaming;
}

hipError_t launch_vocab_pass(const VocabPassArgs& args, bool is_bf16, bool sample,
                             void* workspace, size_t workspace_bytes, hipStream_t stream)
{
    VocabPassArgs a = args;
    // Groups ride along only in a launch of whole rows that has a workgroup for each of them;
    // otherwise they get their own launch first.
    auto separate_advantages = [&]() -> hipError_t {
        const hipError_t err = launch_grpo_advantages(a.adv_rewards, a.adv_offsets, a.adv_groups,
                                                      a.adv_ddof, a.adv_eps, a.adv_out, stream);
        a.adv_groups = 0;
        return err;
    };
    if (a.adv_groups > 0 && a.rows == 0) return separate_advantages();
    if (a.rows == 0) return hipSuccess;
    bool few = false;
    const LaunchPlan whole = vocab_pass_plan(a.rows, a.V, is_bf16, sample, &few);
    if (few && workspace != nullptr && (reinterpret_cast<uintptr_t>(workspace) & 15u) == 0) {
        const SplitPlan plan = split_plan(a.rows, a.V, is_bf16);
        if ((size_t)a.rows * plan.nslots * sizeof(RowPartial) <= workspace_bytes) {
            RowPartial* ws = static_cast<RowPartial*>(workspace);
            if (a.adv_groups > 0) {
                const hipError_t err = separate_advantages();
                if (err != hipSuccess) return err;
            }
            if (is_bf16)
                return sample ? launch_split<ChunkBf16, true>(a, ws, plan, stream)
                              : launch_split<ChunkBf16, false>(a, ws, plan, stream);
            return sample ? launch_split<ChunkF32, true>(a, ws, plan, stream)
                          : launch_split<ChunkF32, false>(a, ws, plan, stream);
        }
    }
    if (a.adv_groups > 0 && (sample || a.adv_groups > whole.workgroups)) {
        const hipError_t err = separate_advantages();
        if (err != hipSuccess) return err;
    }
    if (is_bf16)
        return sample ? launch_for<ChunkBf16, true>(a, whole, stream)
                      : launch_for<ChunkBf16, false>(a, whole, stream);
    return sample ? launch_for<ChunkF32, true>(a, whole, stream)
                  : launch_for<ChunkF32, false>(a, whole, stream);
}

// ---------------------------------------------------------------------------
// Library-owned scratch for callers that cannot allocate: the small-batch path's row
// partials in a file-scope device array instead of a caller workspace.  Every GPU the
// library runs on holds its own copy of the array at its own address, looked up once
// per device; host code uses that address, never the array's name.
// ---------------------------------------------------------------------------
constexpr size_t kStaticScratchBytes = (size_t)kSplitMaxRows * 64 * sizeof(RowPartial);   // 2 MiB
static_assert(kStaticScratchBytes == 2u * 1024 * 1024, "documented size");
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mutex;
static void* g_scratch_ptr[kMaxDevices] = {};

int64_t static_scratch_max_rows() { return kSplitMaxRows; }

hipError_t static_scratch(void** ptr_out, size_t* bytes_out)
{
    int dev = -1;
    hipError_t err = hipGetDevice(&dev);
    if (err != hipSuccess) return err;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (g_scratch_ptr[dev] == nullptr) {
        void* p = nullptr;
        err = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));     // this device's copy
        if (err != hipSuccess) return err;
        if (p == nullptr) return hipErrorInvalidSymbol;
        g_scratch_ptr[dev] = p;
    }
    *ptr_out = g_scratch_ptr[dev];
    *bytes_out = kStaticScratchBytes;
    return hipSuccess;
}

hipError_t launch_entropy_reduce(const float* entropy, const float* gap, const uint8_t* mask, int64_t rows,
                                 double* sum_out, double* gap_sum_out, int64_t* count_out,
                                 hipStream_t stream, hipEvent_t stop_event)
{
    auto kernel = gap_sum_out != nullptr
        ? (mask != nullptr ? entropy_reduce_kernel<true, true> : entropy_reduce_kernel<true, false>)
        : (mask != nullptr ? entropy_reduce_kernel<false, true> : entropy_reduce_kernel<false, false>);
    if (stop_event != nullptr)
        hipExtLaunchKernelGGL(kernel, dim3(1), dim3(1024), 0u, stream, (hipEvent_t) nullptr, stop_event, 0u,
                              entropy, gap, mask, rows, sum_out, gap_sum_out, count_out);
    else
        hipLaunchKernelGGL(kernel, dim3(1), dim3(1024), 0, stream,
                           entropy, gap, mask, rows, sum_out, gap_sum_out, count_out);
    return hipGetLastError();
}

}  // namespace e3
