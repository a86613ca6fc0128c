// Restricted (top-k, optionally followed by top-p) sampling for small k, bf16 and fp32
// rows, for gfx950.
//
// Paper: arXiv 2505.18573 samples its rollouts unrestricted at temperature tau (Section
// 5.1); the truncations are the library's own definition, stated in include/e3.h on value
// LEVELS (the columns that store one bit pattern).  restricted.hip implements it for bf16
// rows through a histogram of all 65,536 patterns; that costs one LDS atomic per column and
// cannot hold the 2^32 patterns of fp32.  For top_k <= 256 the kept set is tiny, and this
// file finds it by selection instead:
//   1. the row is streamed once.  Every thread keeps the maximum of what it has read; a
//      value theta that at least k of these maxima reach is a lower bound of the k-th
//      largest column (k different threads hold a column at or above it), whatever part of
//      the row has been read so far, and it only rises.  Vectors that hold a value at or above
//      the current theta go into a list in LDS (the first requests, which are spread over
//      the whole row, wait in registers for the first theta);
//   2. the columns at or above the final theta are taken from the listed vectors into a list of
//      (key, column); an exact radix select over them gives kappa, the value of the cut
//      level, with the number of columns above it (fewer than k) and on it;
//   3. the columns above kappa are listed, sorted by (value, column), grouped into levels
//      with their fp64 masses, cut by top-p, raced and the winning level's pos-th column
//      taken, exactly as the definition says; the cut level takes part with its count.
// While theta is a plateau that fills most of what a wave holds (zeros, masked columns), only the
// vectors above it are listed, which suffices if the final theta is higher.  If it is not, or the list of vectors
// overflows (values that climb along the row), theta becomes the tightest bound there is, the k-th
// largest of all threads' maxima, and if need be the list is made once more from a second read.  If it overflows
// again (large plateaus of equal values at the cut), every step reads the row instead: slow, same
// results.  100 x 128,000 with 0.13 % of the columns above zeros, top-k 50, all vectors of the
// plateau listed first / so: bf16 158 / 21 us, fp32 202 / 32 us (ordinary rows 17 and 24 us);
// 512 x 151,936 bf16 rows sorted by value 142 / 50 us, fp32 108 / 102 us.
// Every count is exact and every mass fp64, as in restricted.hip.
// Steps 2 (from the radix select on) and 3 exist twice: for any list, with a barrier after
// every short phase, and - for a list of at most 256 candidates and top_k <= 64, the usual
// case - by ranking the list outright (finish_short_list below).
#include "vocab_common.h"
#include "vocab_pass.h"
#include "wave_scan.h"

namespace e3 {
namespace {

constexpr int kSBatch = 8;              // 16-byte requests of a thread made together.  (Two sets of registers; as compiled, a set has
                                       // arrived whole before the next is asked for, which is in flight while it is worked through)
constexpr int kSMaxWaves = 16;
constexpr int kSVecCap = 2688;          // vectors listed in LDS (what two workgroups per compute unit leave room for)
constexpr int kSMaxK = 256;             // top_k served here; the gt-list holds at most kSMaxK - 1 columns
constexpr int kSEqCap = 64;             // columns of the cut level listed for a direct pick
constexpr int kSListCap = 2048;         // candidates (columns at or above theta) listed in LDS
constexpr uint32_t kKeyPosZero = 0x80000000u, kKeyNegZero = 0x7FFFFFFFu;

// Monotone map of a binary32 pattern to an unsigned key (value order, -0 just below +0);
// patterns that are not finite numbers get key 0, below every level.
__device__ __forceinline__ uint32_t key_of_f32(uint32_t bits)
{
    if ((bits & 0x7F800000u) == 0x7F800000u) return 0u;
    return (bits & 0x80000000u) ? ~bits : (bits | 0x80000000u);
}
__device__ __forceinline__ uint32_t f32_of_key(uint32_t key)
{
    return (key & 0x80000000u) ? (key & 0x7FFFFFFFu) : ~key;
}

// The smallest value above a finite one (both zeros are one).
__device__ __forceinline__ float next_above(float z)
{
    const uint32_t b = __float_as_uint(z);
    return __uint_as_float(z > 0.0f ? b + 1u : z < 0.0f ? b - 1u : 1u);
}

// Element access for the two logit types.  A vector is 16 bytes.  Keys are 32-bit; the lower 16
// bits of a bf16 value's key are all ones or all zeros.
struct SelBf16 {
    static constexpr int kElems = 8;
    static constexpr int kKeyBits = 16;              // significant key bits, from the top
    static __device__ __forceinline__ uint32_t elem_bits(const u32x4& v, int j)   // as binary32
    {
        const uint32_t w = j < 2 ? v.x : j < 4 ? v.y : j < 6 ? v.z : v.w;
        return (j & 1) ? (w & 0xFFFF0000u) : (w << 16);
    }
    // columns from `n` on (1 <= n < kElems) replaced by patterns that are not numbers
    static __device__ __forceinline__ u32x4 cut_off(const u32x4& v, int n)
    {
        auto word = [&](uint32_t w, int first) -> uint32_t {
            return n <= first ? 0x7FC07FC0u : n == first + 1 ? (w & 0xFFFFu) | 0x7FC00000u : w;
        };
        return u32x4{word(v.x, 0), word(v.y, 2), word(v.z, 4), word(v.w, 6)};
    }
    static __device__ __forceinline__ uint32_t pattern_of_bits(uint32_t bits) { return bits >> 16; }
    // The largest value where that is not negative: as signed 16-bit integers the patterns of non-negative values are in
    // value order, above those of all others.  Something negative, or no number, where it is negative.
    static __device__ __forceinline__ float quick_max(const u32x4& v)
    {
        typedef int16_t s16x2 __attribute__((ext_vector_type(2)));
        auto halves = [](uint32_t w) { return __builtin_bit_cast(s16x2, w); };
        const s16x2 m = __builtin_elementwise_max(__builtin_elementwise_max(halves(v.x), halves(v.y)),
                                                  __builtin_elementwise_max(halves(v.z), halves(v.w)));
        const uint32_t w = __builtin_bit_cast(uint32_t, m);
        const int hi = (int)w, lo = (int)(w << 16);
        return __uint_as_float((uint32_t)(hi > lo ? hi : lo) & 0xFFFF0000u);
    }
    static __device__ __forceinline__ float vec_max(const u32x4& v)
    {
        return fmax3(fmax3(__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xFFFF0000u), __uint_as_float(v.y << 16)),
                     fmax3(__uint_as_float(v.y & 0xFFFF0000u), __uint_as_float(v.z << 16), __uint_as_float(v.z & 0xFFFF0000u)),
                     fmaxf(__uint_as_float(v.w << 16), __uint_as_float(v.w & 0xFFFF0000u)));
    }
};
struct SelF32 {
    static constexpr int kElems = 4;
    static constexpr int kKeyBits = 32;
    static __device__ __forceinline__ uint32_t elem_bits(const u32x4& v, int j)
    {
        return j == 0 ? v.x : j == 1 ? v.y : j == 2 ? v.z : v.w;
    }
    static __device__ __forceinline__ u32x4 cut_off(const u32x4& v, int n)
    {
        return u32x4{v.x, n <= 1 ? 0x7FC00000u : v.y, n <= 2 ? 0x7FC00000u : v.z, 0x7FC00000u};
    }
    static __device__ __forceinline__ uint32_t pattern_of_bits(uint32_t bits) { return bits; }
    static __device__ __forceinline__ float vec_max(const u32x4& v)
    {
        return fmax3(fmax3(__uint_as_float(v.x), __uint_as_float(v.y), __uint_as_float(v.z)),
                     __uint_as_float(v.w), __uint_as_float(v.w));
    }
};

struct alignas(16) SelShared {
    uint32_t hist[256];
    uint32_t prefix, k_rem, n_eq_last;      // radix select state
    uint32_t n_total;                        // candidates seen by the first pass
    int gt_n, eq_n, list_n, vec_n;           // list fills
    uint32_t skipped;                        // key of the highest plateau of which a wave listed only what lies above (0: none)
    uint32_t k23;                            // the noise word that picks a level's column, 23 bits of it
    uint32_t pad_[2];                        // keeps the arrays below on 16-byte boundaries
    int rank[kSMaxK];
    uint32_t gt_key[kSMaxK];                 // unsorted, then sorted by (key desc, col asc)
    int32_t gt_col[kSMaxK];
    uint32_t st_key[kSMaxK];
    int32_t st_col[kSMaxK];
    double st_M[kSMaxK];                     // inclusive prefix mass in sorted order
    int32_t eq_col[kSEqCap];
    int cut_index;                           // last kept entry of the sorted list (-1: none), or kSMaxK: cut level kept
    float wave_q[kSMaxWaves];
    int wave_lvl[kSMaxWaves];
    int wave_hits[kSMaxWaves];
    int token;
    uint32_t tmax_wave[kSMaxWaves];
};

static_assert(offsetof(SelShared, gt_key) % 16 == 0 && offsetof(SelShared, gt_col) % 16 == 0, "read four at a time");

__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v)
{
    auto most = [&](auto c, auto m) {
        const uint32_t o = (uint32_t)dpp_i<decltype(c)::value, decltype(m)::value>((int)v, (int)v);
        v = o > v ? o : v;
    };
    std::integral_constant<int, 0xF> every;
    most(std::integral_constant<int, kDppXor1>{}, every); most(std::integral_constant<int, kDppXor2>{}, every);
    most(std::integral_constant<int, kDppHalfMirror>{}, every); most(std::integral_constant<int, kDppMirror>{}, every);
    most(std::integral_constant<int, kDppBcast15>{}, std::integral_constant<int, 0xA>{});
    most(std::integral_constant<int, kDppBcast31>{}, std::integral_constant<int, 0xC>{});
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// One 8-bit pass of a radix select for the k-th largest: every thread has added its keys
// that match `prefix` above `shift + 8` to hist; wave 0 finds the digit that holds rank k_rem.
__device__ __forceinline__ void select_digit(SelShared& sh, int tid)
{
    if (tid < 64) {
        // lane l owns bins 255 - 4l .. 252 - 4l (descending)
        uint32_t c[4], sum = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) { c[j] = sh.hist[255 - 4 * tid - j]; sum += c[j]; }
        const uint32_t inc = (uint32_t)wave_prefix_sum((int)sum);
        uint32_t before = inc - sum;                       // counts in higher bins
        const uint32_t k = sh.k_rem;
        if (before < k && k <= inc) {                       // exactly one lane
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (before < k && k <= before + c[j]) {
                    sh.prefix = (sh.prefix << 8) | (uint32_t)(255 - 4 * tid - j);
                    sh.k_rem = k - before;
                    sh.n_eq_last = c[j];
                    before = 0xFFFFFFFFu;                   // done
                } else if (before != 0xFFFFFFFFu) {
                    before += c[j];
                }
            }
        }
    }
}

struct SelArgs {
    const void* logits;
    int64_t rows, V, row_stride;
    const float* tau_rows;
    float tau_scalar;
    int32_t top_k;
    float top_p;
    uint64_t seed, row_base;
    int32_t* token_out;
    float* logp_out;
    int32_t* kept_out;
};

// ---------------------------------------------------------------------------
// The rest of a row for a short candidate list (at most kSoloList entries in LDS) and a small
// count cut (top_k <= kSoloK): the usual case.  Same definition and arithmetic as the workgroup-wide
// code in the kernel below, in three steps with two barriers.  What bounds it is the number of
// dependent instructions of a wave, so everything that can be done per candidate is done by all waves at once:
//   rank    the list is ranked as it is, the L x L comparisons spread over the waves (a group of 64 entries against one
//           part of the others each); one of them also draws the entries' race noise, another takes the fp64
//           exponentials.  The k-th largest needs no search: it is the entry of rank k - 1;
//   sort    entries go to their rank, equal values in any order (the pick below orders a level's columns);
//   finish  one wave, one sorted entry per lane: levels, masses, cuts, race and pick are scans, ballots and
//           lane reads.  Fewer than k <= 64 entries stand above the cut level and its first one stands
//           behind them, so 64 lanes see all that matters; the rest of the cut level is only counted.
// 512 rows x 151,936 bf16 columns, top-k 50 (lists of 70 to 190): one wave alone that searched the k-th largest bit by bit
// (1500 cycles, 4000 for fp32) and ranked the columns above it through lane broadcasts (4000) took 10,200 cycles, these
// steps take 4900.  64 rows x 32,000, top-k 50: bf16 10.7 -> 8.4 us, fp32 11.5 -> 8.3 us.
// ---------------------------------------------------------------------------
constexpr int kSoloList = 256;
constexpr int kSoloK = 64;

// How many of four keys are above `key`, added to two counters: two instructions a key.  Written as asm because the compiler
// puts a comparison right before the addition that takes its result as a carry, which this part makes wait; here three
// instructions stand between them (two are needed).
__device__ __forceinline__ void count_above(int& n0, int& n1, const uint4& o, uint32_t key)
{
    uint64_t c0, c1, c2, c3;
    asm("v_cmp_gt_u32_e64 %2, %6, %10\n\t"
        "v_cmp_gt_u32_e64 %3, %7, %10\n\t"
        "v_cmp_gt_u32_e64 %4, %8, %10\n\t"
        "v_cmp_gt_u32_e64 %5, %9, %10\n\t"
        "v_addc_co_u32_e64 %0, vcc, 0, %0, %2\n\t"
        "v_addc_co_u32_e64 %1, vcc, 0, %1, %3\n\t"
        "v_addc_co_u32_e64 %0, vcc, 0, %0, %4\n\t"
        "v_addc_co_u32_e64 %1, vcc, 0, %1, %5"
        : "+v"(n0), "+v"(n1), "=&s"(c0), "=&s"(c1), "=&s"(c2), "=&s"(c3)
        : "v"(o.x), "v"(o.y), "v"(o.z), "v"(o.w), "v"(key) : "vcc");
}

// LDS of these steps that other steps use as well: SelShared::rank holds the ranks, gt_col counts the entries sent to a rank
// (both zeroed when the kernel starts, as are the first kSoloList keys of the list), st_key and st_col are the
// sorted list, st_M its weights and gt_key its noise; `mass` and `noise` (kSoloList each) are the same before sorting.
template <typename T, int kSThreads>
__device__ __forceinline__ void finish_short_list(const SelArgs& a, SelShared& sh, const uint32_t* lkey,
                                                  const int32_t* lcol, double* mass, float* noise, int n_list,
                                                  int k_req, int64_t row, uint64_t grow, double inv_tau, float c,
                                                  int lane, int wave)
{
    constexpr int kSWaves = kSThreads / 64;
    constexpr int kLgWaves = kSWaves == 16 ? 4 : 3;
    static_assert(kSWaves == 1 << kLgWaves && kSoloList == 256, "whole parts, at least two");
    const int lg_groups = n_list <= 64 ? 0 : n_list <= 128 ? 1 : 2;
    const int groups = 1 << lg_groups, parts = kSWaves >> lg_groups;
    const int group = wave & (groups - 1), part = wave >> lg_groups;
    const int entry = group * 64 + lane;                            // (keys behind the list are 0: below every real one)
    const uint32_t key = lkey[entry];
    const bool mine = entry < n_list;

    // ---- rank: the entries above mine, among my part of the list; the last two parts of four or more have other work
    const int lg_rank = parts == 2 ? 1 : parts == 4 ? 1 : parts == 8 ? 2 : 3;
    if (part < 1 << lg_rank) {
        const int per = (((n_list - 1) >> lg_rank) + 16) & ~15;      // a multiple of the sixteen entries read together
        const int end = (part + 1) * per < n_list ? (part + 1) * per : n_list;
        int above = 0, above1 = 0;
        for (int e = part * per; e < end; e += 16) {
            uint4 o[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) o[u] = reinterpret_cast<const uint4*>(&lkey[e])[u];
#pragma unroll
            for (int u = 0; u < 4; ++u) count_above(above, above1, o[u], key);
        }
        above += above1;
        if (mine && above != 0) atomicAdd(&sh.rank[entry], above);
    }
    if (part == parts - 1) {
        // race noise of the level: E_j from Philox stream 3 at the level's stored pattern
        const uint32_t pat = T::pattern_of_bits(f32_of_key(key));
        uint32_t w4[4];
        philox4x32_10(pat >> 2, (uint32_t)grow, (uint32_t)(grow >> 32), 3u,
                      (uint32_t)a.seed, (uint32_t)(a.seed >> 32), w4);
        const int sel = pat & 3;
        noise[entry] = inv_exp_variate(sel == 0 ? w4[0] : sel == 1 ? w4[1] : sel == 2 ? w4[2] : w4[3]);
    } else if (part == parts - 2) {
        // weights relative to the row's largest column, which every list holds
        uint32_t top = 0u;
        for (int e = lane; e < groups * 64; e += 64) top = lkey[e] > top ? lkey[e] : top;
        top = wave_max_u32(top);
        const double z1 = (double)__uint_as_float(f32_of_key(top));
        mass[entry] = exp(((double)__uint_as_float(f32_of_key(key)) - z1) * inv_tau);
    }
    __syncthreads();

    // ---- sort
    if (wave < groups && mine) {
        const int r = sh.rank[entry];
        const int at = r + atomicAdd(&sh.gt_col[r], 1);
        sh.st_key[at] = key;
        sh.st_col[at] = lcol[entry];
        sh.st_M[at] = mass[entry];
        sh.gt_key[at] = __float_as_uint(noise[entry]);
    }
    __syncthreads();
    if (wave != 0) return;

    // ---- finish: lane = rank
    const bool real = lane < n_list;
    const uint32_t skey = real ? sh.st_key[lane] : 0u;
    const int32_t scol = real ? sh.st_col[lane] : 0;
    const double w = real ? sh.st_M[lane] : 0.0;
    const float inv_e = __uint_as_float(sh.gt_key[lane]);           // read for real entries only
    const int k_eff = n_list < k_req ? n_list : k_req;              // fewer than k finite columns: all of them
    const uint32_t kappa = (uint32_t)__builtin_amdgcn_readlane((int)skey, k_eff - 1);
    const int n = (int)__popcll(__ballot(real && skey > kappa));    // columns above the cut level: lanes 0 .. n - 1; lane n is its first
    int n_cut = (int)__popcll(__ballot(real && skey == kappa));
    if (__builtin_amdgcn_readlane((int)skey, 63) == (int)kappa)     // (a list of fewer than 64 ends with key 0)
        for (int e = 64 + lane; e < groups * 64; e += 64) n_cut += (int)__popcll(__ballot(e < n_list && sh.st_key[e] == kappa));

    // masses in rank order (fp64), cuts
    const uint32_t key1 = (uint32_t)__builtin_amdgcn_readlane((int)skey, 0);       // the row's highest level
    const double z1 = (double)__uint_as_float(f32_of_key(key1));
    const double M = wave_prefix_sum(lane < n ? w : 0.0);           // inclusive prefix mass
    const double M_gt = n > 0 ? read_lane(M, n - 1) : 0.0;
    const double M_k = M_gt + (double)n_cut * read_lane(w, n);      // mass of the top-k set
    constexpr int kNextLane = 0x130, kPrevLane = 0x138;             // wave_shl:1, wave_shr:1
    const uint32_t next_key = (uint32_t)dpp_i<kNextLane>(0, (int)skey);
    const uint32_t prev_key = (uint32_t)dpp_i<kPrevLane>(0, (int)skey);
    int kept_sorted = n + 1;                                        // lanes of kept levels (the cut level in lane n) ...
    int kept_C = n + n_cut;                                         // ... and their columns: by default down to the cut level
    double M_kept = M_k;
    if (a.top_p < 1.0f) {
        // top-p on the renormalised top-k set: first level end whose cumulative mass reaches the target
        const double Tm = (double)a.top_p * M_k;
        const bool level_end = lane < n && next_key != skey;        // (lane n's key differs from lane n - 1's)
        const unsigned long long reach = __ballot(level_end && M >= Tm);
        if (reach != 0ull) {
            const int cut_index = (int)__builtin_ctzll(reach);
            kept_sorted = kept_C = cut_index + 1;
            M_kept = read_lane(M, cut_index);
        }
    }
    const double ln_M = log(M_kept);

    // race of the kept levels, each scored by its first lane
    const bool level_start = lane <= n && (lane == 0 || prev_key != skey);
    const unsigned long long starts = __ballot(level_start);
    const unsigned long long later = lane < 63 ? starts >> (lane + 1) : 0ull;
    const int cnt = lane == n ? n_cut : 1 + (int)__builtin_ctzll(later | 1ull << 63);     // columns of my level
    const float z1f = __uint_as_float(f32_of_key(key1));
    float my_q = -1.0f;
    if (level_start && lane < kept_sorted)
        my_q = (float)cnt * __builtin_amdgcn_exp2f((__uint_as_float(f32_of_key(skey)) - z1f) * c) * inv_e;
    const float best_q = wave_max(my_q);
    const unsigned long long winners = __ballot(my_q == best_q);
    const int best = (int)__builtin_ctzll(winners | 1ull << 63);    // ties: the higher level

    // the column inside the winning level: the pos-th of its columns
    int tok = 0;
    uint32_t tok_key = key1;
    if (best_q >= 0.0f) {
        tok_key = (uint32_t)__builtin_amdgcn_readlane((int)skey, best);
        const int level_cnt = __builtin_amdgcn_readlane(cnt, best);
        tok = __builtin_amdgcn_readlane(scol, best);
        if (level_cnt > 1) {
            const int pos = (int)(((2u * (uint64_t)sh.k23 + 1u) * (uint64_t)level_cnt) >> 24);
            for (int e0 = 0; e0 < level_cnt; e0 += 64) {
                const int e = e0 + lane;
                const int32_t mc = e < level_cnt ? sh.st_col[best + e] : 0x7FFFFFFF;
                int before = 0;
                for (int f = 0; f < level_cnt; ++f) before += sh.st_col[best + f] < mc;
                const unsigned long long hit = __ballot(e < level_cnt && before == pos);
                if (hit != 0ull) tok = __builtin_amdgcn_readlane(mc, (int)__builtin_ctzll(hit));
            }
        }
    }
    if (lane == 0) {
        if (tok < 0 || tok >= a.V) tok = 0;
        a.token_out[row] = tok;
        if (a.kept_out) a.kept_out[row] = kept_C;
        if (a.logp_out)
            a.logp_out[row] = best_q >= 0.0f
                ? (float)(((double)__uint_as_float(f32_of_key(tok_key)) - z1) * inv_tau - ln_M)
                : __builtin_nanf("");
    }
}

// Bound by the read of the row plus ~3.5 us of short dependent phases after it.  512 threads per row,
// two workgroups per compute unit (one row's short phases overlap the other's stream) and
// non-temporal loads, or 1024 threads and plain loads for at most one row per compute unit (half the
// stream's latency; such a batch may sit in the caches: 100 fp32 rows 24.7 us plain, 28.2 us
// non-temporal; 300 rows x 151,936 bf16 29.7 us with 512 threads, 48 us with 1024): four waves per
// SIMD and up to 128 vector registers either way.  151,936 bf16 columns, top-k 50 + top-p 0.95: 8 rows 13.1 us,
// 512 rows 30.0 us (5.2 TB/s), 1024 rows 52.8 us (5.9 TB/s); with one wave finishing a row alone (see finish_short_list)
// and the candidates taken column by column from the listed vectors 16.5, 33.7 and 59.6.
template <typename T, int kSThreads>
__global__ __launch_bounds__(kSThreads) __attribute__((amdgpu_waves_per_eu(4, 4)))
void sample_select_kernel(SelArgs a)
{
    constexpr int kSWaves = kSThreads / 64;
    constexpr bool kStream = kSThreads == 512;
    static_assert(kSWaves <= kSMaxWaves, "one slot per wave");
    __shared__ u32x4 lvec[kSVecCap];                              // listed vectors and their indices
    __shared__ int32_t lvec_at[kSVecCap];
    __shared__ uint32_t lkey[kSListCap];                          // candidate columns
    __shared__ int32_t lcol[kSListCap];
    __shared__ SelShared sh;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t row = blockIdx.x;
    const int64_t V = a.V;
    const int esz = 16 / T::kElems;
    const char* rowp = static_cast<const char*>(a.logits) + row * a.row_stride * esz;
    const u32x4* rv = reinterpret_cast<const u32x4*>(rowp);
    // the last vector may reach past V (inside the row pitch)
    const int nvec = (int)((V + T::kElems - 1) / T::kElems);
    const int last = (int)(V - (int64_t)(nvec - 1) * T::kElems);  // its columns, 1 .. kElems
    const float tau = a.tau_rows ? a.tau_rows[row] : a.tau_scalar;
    const double inv_tau = 1.0 / (double)tau;
    const float c = kLog2eF / tau;
    const uint64_t grow = a.row_base + (uint64_t)row;
    const int k_req = a.top_k < kSMaxK ? a.top_k : kSMaxK;

    // ---- 1. the stream ----------------------------------------------------------------------
    // Slot s of a thread is vector tid + kSThreads s; a set of requests takes every nsets-th slot, so
    // that each set, above all the first, samples the whole row.
    const int nslots = (nvec + kSThreads - 1) / kSThreads;
    const int whole = (int)(V / T::kElems) / kSThreads;           // slots of nothing but complete vectors
    const int nsets = (nslots + kSBatch - 1) / kSBatch;
    const u32x4 none = {0x7FC07FC0u, 0x7FC07FC0u, 0x7FC07FC0u, 0x7FC07FC0u};   // no numbers, as bf16 and as fp32
    auto guarded = [&](int v) -> u32x4 {
        u32x4 x = none;
        if (v < nvec) x = rv[v];
        if (v == nvec - 1 && last < T::kElems) x = T::cut_off(x, last);
        return x;
    };
    // Requests never branch: a load on one side of a branch makes the compiler wait for it where the sides
    // meet.  Past the row they repeat its last vector, whose maximum then does not count.
    auto request = [&](u32x4 (&x)[kSBatch], int set) {
#pragma unroll
        for (int u = 0; u < kSBatch; ++u) {
            const int v = tid + (set + u * nsets) * kSThreads;
            const uint32_t at = (uint32_t)(v < nvec ? v : nvec - 1) * 16u;
            const u32x4* p = reinterpret_cast<const u32x4*>(rowp + at);
            x[u] = kStream ? stream_load(p) : *p;
        }
    };
    float tmax = -INFINITY;                                       // maximum of the finite values I have read
    // Maxima are taken as floats (NaN operands drop out of v_max3); a vector whose maximum is
    // infinite is looked through by hand.
    auto finite_max = [&](u32x4 x) -> float {
        asm volatile("" : "+v"(x));                               // shares nothing with the common path, which would hold it in registers
        float f = -INFINITY;
#pragma unroll
        for (int j = 0; j < T::kElems; ++j) {
            const float z = __uint_as_float(T::elem_bits(x, j));
            f = z < INFINITY ? fmaxf(f, z) : f;
        }
        return f;
    };
    auto past_the_end = [&](const u32x4 (&x)[kSBatch], float (&m)[kSBatch], int set) {
#pragma unroll
        for (int u = 0; u < kSBatch; ++u) {
            const int slot = set + u * nsets;
            if (slot >= whole) {                                  // uniform: holds the row's end or lies past it
                const int v = tid + slot * kSThreads;
                if (v >= nvec) m[u] = -INFINITY;
                else if (v == nvec - 1 && last < T::kElems) m[u] = finite_max(T::cut_off(x[u], last));
            }
        }
    };
    // bf16 rows that have a compute unit each: the maxima of a set as quick_max leaves them suffice while every lane has a value
    // that is not negative among its vectors and theta is above zero: then none of those that it gets wrong reaches theta.  Else the
    // exact ones, from then on (`by_value`, wave-uniform), and from the start for a row of one set, which could not earn back a
    // second look, and where a wave's first request holds negative columns only (log-probabilities, masks).  With
    // two rows to a compute unit exact maxima only: both in every set, as the branch there would make the compiler wait for the set in
    // flight, cost rows that are negative throughout more than the others gained (quick first / exact, us: 512 x 151,936
    // ordinary 29.8 / 30.0, log-probabilities 32.3 / 30.2; 300 x 70,005 17.7 / 18.1 and 19.8 / 17.9; 300 x 1000 of one set, top-k 50,
    // 11.1 / 9.8).
    constexpr bool kQuick = T::kKeyBits == 16 && !kStream;
    bool by_value = !kQuick;
    auto exact_maxima = [&](const u32x4 (&x)[kSBatch], float (&m)[kSBatch], int set) {
        float most = -INFINITY;
#pragma unroll
        for (int u = 0; u < kSBatch; ++u) { m[u] = T::vec_max(x[u]); most = fmaxf(most, m[u]); }
        if (__builtin_expect(__any(most == INFINITY), 0)) {
#pragma unroll
            for (int u = 0; u < kSBatch; ++u) m[u] = finite_max(x[u]);
        }
        past_the_end(x, m, set);
    };
    auto set_maxima = [&](const u32x4 (&x)[kSBatch], float (&m)[kSBatch], int set) {
        if constexpr (kQuick) {
            if (!by_value) {
                float most = -INFINITY;
#pragma unroll
                for (int u = 0; u < kSBatch; ++u) m[u] = T::quick_max(x[u]);
                past_the_end(x, m, set);
                // (no numbers of a positive sign are above infinity as integers, and drop out of `most` as floats: looked for one by one)
                bool odd = false;
#pragma unroll
                for (int u = 0; u < kSBatch; ++u) { most = fmaxf(most, m[u]); odd |= m[u] != m[u]; }
                by_value = __any(odd || !(most >= 0.0f && most < INFINITY));
            }
            if (__builtin_expect(by_value, 0)) exact_maxima(x, m, set);
        } else {
            exact_maxima(x, m, set);
        }
    };
    // The wave's m-th largest thread maximum, m = ceil(k / waves with columns), bit by bit from the
    // top with one ballot per bit: the largest value that at least m lanes reach.  The upper 16 bits
    // settle an ordinary row; the lower ones of an fp32 row count only where more than m lanes share the
    // upper ones, i.e. for values that differ by little of themselves (8 rows x 151,936 of
    // 100 + 0.3 N(0, 1), top-k 50: 125 us with 16 bits, when the list of vectors overflows twice, 23.5 us so).
    // The smallest of the waves' values has waves x m >= k threads at or above it.  Values
    // published earlier are lower bounds as well: no barrier between a refinement and its readers.
    const int full_waves = nvec / 64 < 1 ? 1 : nvec / 64 < kSWaves ? nvec / 64 : kSWaves;
    const int m_th = (k_req + full_waves - 1) / full_waves;
    auto publish = [&]() {
        if (wave >= full_waves) return;
        const uint32_t key = tmax == 0.0f ? kKeyPosZero : key_of_f32(__float_as_uint(tmax));
        uint32_t wm = 0u;
        for (int b = 31; b >= 16; --b) {
            const uint32_t cand = wm | (1u << b);
            if ((int)__popcll(__ballot(key >= cand)) >= m_th) wm = cand;
        }
        if (T::kKeyBits > 16 && (int)__popcll(__ballot(key >= wm)) > m_th) {
            // the m-th largest is among the lanes that share its upper bits: one of them after the other as
            // pivot, each step drops it and all lanes on the wrong side of it (equal values: one step)
            unsigned long long open = __ballot((key >> 16) == (wm >> 16));
            for (;;) {
                const uint32_t v = (uint32_t)__builtin_amdgcn_readlane((int)key, (int)__builtin_ctzll(open));
                const unsigned long long ge = __ballot(key >= v), gt = __ballot(key > v);
                if ((int)__popcll(gt) >= m_th) open &= gt;
                else if ((int)__popcll(ge) < m_th) open &= ~ge;
                else { wm = v; break; }
            }
        }
        if (lane == 0) __hip_atomic_store(&sh.tmax_wave[wave], wm, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    };
    auto current_theta = [&]() -> uint32_t {
        uint32_t t = lane < full_waves ? __hip_atomic_load(&sh.tmax_wave[lane & (kSWaves - 1)], __ATOMIC_RELAXED,
                                                        __HIP_MEMORY_SCOPE_WORKGROUP) : 0xFFFFFFFFu;
        // sixteen lanes hold them
        auto least = [&](auto c) { const uint32_t o = (uint32_t)dpp_i<decltype(c)::value>((int)t, (int)t); t = o < t ? o : t; };
        least(std::integral_constant<int, kDppXor1>{}); least(std::integral_constant<int, kDppXor2>{});
        least(std::integral_constant<int, kDppHalfMirror>{}); least(std::integral_constant<int, kDppMirror>{});
        t = (uint32_t)__builtin_amdgcn_readfirstlane((int)t);
        if (t == 0u) t = 1u;                                      // a wave with fewer than m finite maxima: every finite value
        // a zero maximum was recorded as +0 whichever zero it was: let -0 in as well
        return t == kKeyPosZero ? kKeyNegZero : t;
    };
    auto theta_value = [&](uint32_t t) -> float {                 // as a value to compare with (keys below the lowest finite one are no numbers)
        const uint32_t bits = f32_of_key(t);                      // (a bf16 value has a low half of zeros)
        return t < 0x00800000u ? -3.402823466e38f : __uint_as_float(T::kKeyBits == 16 ? bits & 0xFFFF0000u : bits);
    };
    // The vectors of a set whose maximum reaches theta go into the list: one reservation per wave, a ballot per request, and
    // nothing for a request without a hit (the stream is bound by its instructions where a row has a compute unit: 8 x 151,936
    // 13.5 us, 14.3 with a prefix sum over the lanes, every request's stores behind its own conditions and floating-point maxima).
    // Where that would be a quarter of the set, theta is a plateau so far, and only what lies above
    // it is listed (sh.skipped remembers the highest such value): enough if the final theta is higher.
    auto list_set = [&](const u32x4 (&x)[kSBatch], float (&m)[kSBatch], int set, float thf, bool all) {
        if (kQuick && __builtin_expect(thf <= 0.0f && !by_value, 0)) {                               // uniform
            by_value = true;
            exact_maxima(x, m, set);
        }
        float bound = thf;
        unsigned long long hit[kSBatch];
        auto count = [&]() -> int {
            int n = 0;
#pragma unroll
            for (int u = 0; u < kSBatch; ++u) { hit[u] = __ballot(m[u] >= bound); n += (int)__popcll(hit[u]); }
            return n;
        };
        int total = count();
        if (total == 0) return;
        if (__builtin_expect(!all && total > 16 * kSBatch, 0)) {
            bound = next_above(thf);
            if (lane == 0) atomicMax(&sh.skipped, key_of_f32(__float_as_uint(thf)));
            total = count();
        }
        int base = 0;
        if (lane == 0) base = atomicAdd(&sh.vec_n, total);
        base = __builtin_amdgcn_readfirstlane(base);
#pragma unroll
        for (int u = 0; u < kSBatch; ++u) {
            if (hit[u] != 0ull) {                                 // uniform
                const int slot = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(hit[u] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)hit[u], (uint32_t)base));
                if (m[u] >= bound && slot < kSVecCap) { lvec[slot] = x[u]; lvec_at[slot] = tid + (set + u * nsets) * kSThreads; }
                base += (int)__popcll(hit[u]);
            }
        }
    };
    if (tid == 0) { sh.gt_n = 0; sh.eq_n = 0; sh.token = 0; sh.list_n = 0; sh.vec_n = 0; sh.skipped = 0u; }
    if (tid < kSoloList) { sh.rank[tid] = 0; sh.gt_col[tid] = 0; lkey[tid] = 0u; }
    {
        u32x4 x[kSBatch], y[kSBatch];
        float m[kSBatch];
        auto maxima = [&](const u32x4 (&x)[kSBatch], int set) {
            set_maxima(x, m, set);
#pragma unroll
            for (int u = 0; u < kSBatch; ++u) tmax = fmaxf(tmax, m[u]);
        };
        request(x, 0);
        // Sixteen waves ask for their second set when the first has come: its requests would stand in line before the last
        // waves' first, which everybody waits for (100 x 128,000 fp32, top-k 20 17.1 -> 16.0 us, 8 x 151,936 13.5 -> 13.1; two
        // rows of eight waves to a compute unit want both in flight, 512 rows 30.4 and 30.0).
        if (kStream && nsets > 1) request(y, 1);
        if (wave == kSWaves - 1) {                                // while they are in flight
            uint32_t w4[4];
            philox4x32_10(0u, (uint32_t)grow, (uint32_t)(grow >> 32), 4u, (uint32_t)a.seed, (uint32_t)(a.seed >> 32), w4);
            if (lane == 0) sh.k23 = w4[0] >> 9;
        }
        if constexpr (kQuick) by_value = nsets == 1 || __all((x[0].x & x[0].y & x[0].z & x[0].w & 0x80008000u) == 0x80008000u);
        maxima(x, 0);
        if (!kStream && nsets > 1) request(y, 1);
        publish();
        // orders LDS only: __syncthreads() would wait for the loads in flight as well
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        float thf = theta_value(current_theta());
        list_set(x, m, 0, thf, nsets == 1);
        // refined whenever what has been read has doubled, and at the end; after every set for a large k, whose list
        // would overflow otherwise (512 x 151,936, top-k 256, a list of 2048 / of 2688 / and refined so: fp32 108 / 89 / 73 us,
        // bf16 54 / 48 / 48; at k = 100 it would cost 0.5 us)
        const bool often = k_req > (kSThreads == 512 ? 160 : 224);
        auto refine = [&](int set) {
            if (set + 1 == nsets || (set & (set + 1)) == 0 || often) { publish(); thf = theta_value(current_theta()); }
        };
        for (int set = 1; set < nsets; set += 2) {
            if (set + 1 < nsets) request(x, set + 1);
            maxima(y, set);
            list_set(y, m, set, thf, nsets == 1);
            refine(set);
            if (set + 1 >= nsets) break;
            if (set + 2 < nsets) request(y, set + 2);
            maxima(x, set + 1);
            list_set(x, m, set + 1, thf, nsets == 1);
            refine(set + 1);
        }
    }
    __syncthreads();
    uint32_t theta = current_theta();
    // The waves' bounds are loose where the large columns are unevenly spread over the waves (few
    // columns stand out of a plateau, or the row is sorted): then the k-th largest of all threads' maxima,
    // bit by bit as in a wave (rare, and kept small).
    auto exact_theta = [&]() -> uint32_t {
        const uint32_t key = tmax == 0.0f ? kKeyPosZero : key_of_f32(__float_as_uint(tmax));
        if (tid < 32) sh.hist[tid] = 0u;
        __syncthreads();
        uint32_t t = 0u;
#pragma unroll 1
        for (int b = 31; b >= 32 - T::kKeyBits; --b) {
            const uint32_t cand = t | (1u << b);
            const uint32_t mine = (uint32_t)__popcll(__ballot(key >= cand));
            if (lane == 0 && mine != 0u) atomicAdd(&sh.hist[b], mine);
            __syncthreads();
            if (sh.hist[b] >= (uint32_t)k_req) t = cand;
        }
        __syncthreads();                                          // sh.hist is used again
        if (t == 0u) t = 1u;                                      // fewer than k finite maxima: every finite value
        return t == kKeyPosZero ? kKeyNegZero : t;
    };
    int n_vec = sh.vec_n;
    const uint32_t skipped = sh.skipped;
    if (__builtin_expect((n_vec > kSVecCap) | (skipped != 0u), 0)) {          // uniform
        // the list suffices for a theta above all that were skipped (as values: the zeros are one)
        const float above = skipped != 0u ? __uint_as_float(f32_of_key(skipped)) : -INFINITY;
        if (n_vec > kSVecCap || !(theta_value(theta) > above)) theta = exact_theta();
        if (n_vec > kSVecCap || !(theta_value(theta) > above)) {
            __syncthreads();
            if (tid == 0) sh.vec_n = 0;
            __syncthreads();
            u32x4 x[kSBatch];
            float m[kSBatch];
            const float thf = theta_value(theta);
#pragma unroll 1
            for (int set = 0; set < nsets; ++set) {
                request(x, set);
                set_maxima(x, m, set);
                list_set(x, m, set, thf, true);
            }
            __syncthreads();
            n_vec = sh.vec_n;
        }
    }

    // ---- 2. the candidates: every finite column whose key reaches theta ----------------------------
    auto stream_candidates = [&](auto&& f) {
        for (int s = 0; s < nslots; ++s) {
            const int v = tid + s * kSThreads;
            const u32x4 x = guarded(v);
#pragma unroll
            for (int e = 0; e < T::kElems; ++e) {
                const uint32_t key = key_of_f32(T::elem_bits(x, e));
                if (key >= theta) f(key, (int32_t)(v * T::kElems + e));
            }
        }
    };
    // one slot per true flag, one LDS atomic per wave instruction
    auto wave_slot = [&](bool flag, int* counter) -> int {
        const unsigned long long m = __ballot(flag);
        if (m == 0ull) return -1;
        int base = 0;
        const int leader = (int)__builtin_ctzll(m);
        if (lane == leader) base = atomicAdd(counter, __popcll(m));
        base = __shfl(base, leader, 64);
        return base + __popcll(m & ((1ull << lane) - 1ull));
    };
    if (n_vec <= kSVecCap) {
        const float thf = theta_value(theta);
        const int32_t vlast = (int32_t)V - T::kElems;                 // vectors beginning behind it are cut short by the row's end
        for (int i0 = 0; i0 < n_vec; i0 += kSThreads) {           // whole waves: the reservation is wave-wide
            const int i = i0 + tid;
            const u32x4 x = lvec[i < n_vec ? i : 0];
            const int32_t col0 = lvec_at[i < n_vec ? i : 0] * T::kElems;
            // as values: a key reaches theta where the value does (zeros: theta is never that of +0), and is finite
            uint32_t hits = 0u;
#pragma unroll
            for (int e = 0; e < T::kElems; ++e) {
                const float z = __uint_as_float(T::elem_bits(x, e));
                hits |= (uint32_t)(z >= thf && z < INFINITY) << e;
            }
            if (col0 > vlast) hits &= (1u << last) - 1u;              // the last vector may reach past the row
            hits = i < n_vec ? hits : 0u;
            const int mine = __popc(hits);
            const int inc = wave_prefix_sum(mine);
            if (__builtin_amdgcn_readlane(inc, 63) == 0) continue;
            int base = 0;
            if (lane == 63) base = atomicAdd(&sh.list_n, inc);
            int slot = __builtin_amdgcn_readlane(base, 63) + inc - mine;
            auto enter = [&](int e) {
                if (slot < kSListCap) { lkey[slot] = key_of_f32(T::elem_bits(x, e)); lcol[slot] = col0 + e; }
                ++slot;
            };
            // a hit at a time: one or two rounds, where the vector's columns one after the other would be as many as it has; but not
            // where a lane has many (sorted rows, a large k, plateaus: bf16 300 x 4000 sorted, top-k 50, 21.5 us column by
            // column, 23.6 a hit at a time, 21.6 so)
            if (!__any(mine > 3)) {
                for (; hits != 0u; hits &= hits - 1u) enter((int)__builtin_ctz(hits));
            } else {
#pragma unroll
                for (int e = 0; e < T::kElems; ++e) {
                    if (hits >> e & 1u) enter(e);
                }
            }
        }
    } else if (tid == 0) {
        sh.list_n = kSListCap + 1;
    }
    __syncthreads();
    const int n_list = sh.list_n;
    if (n_list == 0) {                                            // no finite logit in the row
        if (tid == 0) {
            a.token_out[row] = 0;
            if (a.kept_out) a.kept_out[row] = 0;
            if (a.logp_out) a.logp_out[row] = __builtin_nanf("");
        }
        return;
    }
    const bool listed = n_list <= kSListCap;
    if (n_list <= kSoloList && k_req <= kSoloK) {                  // short list, small k: ranked as it is
        // (the listed vectors are no longer needed)
        double* mass = reinterpret_cast<double*>(lvec);
        finish_short_list<T, kSThreads>(a, sh, lkey, lcol, mass, reinterpret_cast<float*>(mass + kSoloList), n_list, k_req,
                                        row, grow, inv_tau, c, lane, wave);
        return;
    }
    auto for_each_candidate = [&](auto&& f) {
        if (listed) {
            for (int e = tid; e < n_list; e += kSThreads) f(lkey[e], lcol[e]);
        } else if (n_vec <= kSVecCap) {
            for (int i = tid; i < n_vec; i += kSThreads) {
                const u32x4 x = lvec[i];
                const int32_t col0 = lvec_at[i] * T::kElems;
#pragma unroll
                for (int e = 0; e < T::kElems; ++e) {
                    const uint32_t key = key_of_f32(T::elem_bits(x, e));
                    if (col0 + e < V && key >= theta) f(key, col0 + e);
                }
            }
        } else {
            stream_candidates(f);
        }
    };

    // kappa: the k-th largest column (exact), by radix select over the candidates ---------
    if (tid == 0) { sh.prefix = 0u; sh.k_rem = 0u; sh.n_total = 0u; }
    uint32_t k_col = (uint32_t)k_req;
    for (int pass = 0; pass < T::kKeyBits / 8; ++pass) {
        const int shift = 24 - 8 * pass;
        if (tid < 256) sh.hist[tid] = 0u;
        __syncthreads();
        const uint32_t prefix = sh.prefix;
        for_each_candidate([&](uint32_t key, int32_t) {
            if (pass == 0 || (key >> (shift + 8)) == prefix) atomicAdd(&sh.hist[(key >> shift) & 255u], 1u);
        });
        __syncthreads();
        if (pass == 0) {
            // number of candidates; fewer than k finite columns in the row: the cut is the lowest level
            if (tid < 64) {
                const uint32_t t = (uint32_t)wave_prefix_sum((int)(sh.hist[tid] + sh.hist[tid + 64] + sh.hist[tid + 128] + sh.hist[tid + 192]));
                if (tid == 63) { sh.n_total = t; sh.k_rem = t < k_col ? t : k_col; }
            }
            __syncthreads();
        }
        select_digit(sh, tid);
        __syncthreads();
    }
    const uint32_t kappa = T::kKeyBits == 32 ? sh.prefix
                         : ((sh.prefix << 16) | ((sh.prefix & 0x8000u) ? 0u : 0xFFFFu));   // rebuild a bf16 value's key
    const int n_cut = (int)sh.n_eq_last;                          // columns on the cut level
    const uint32_t k_eff = sh.n_total < (uint32_t)k_req ? sh.n_total : (uint32_t)k_req;
    const int count_gt = (int)(k_eff - sh.k_rem);                 // columns above it (< k)
    __syncthreads();

    // ---- 3. the columns above kappa, and those on it when they are few -------------------------------
    if (listed) {
        for (int e0 = 0; e0 < n_list; e0 += kSThreads) {          // whole waves: wave_slot is wave-wide
            const int e = e0 + tid;
            const uint32_t key = e < n_list ? lkey[e] : 0u;
            const int32_t col = e < n_list ? lcol[e] : 0;
            const int sg = wave_slot(key > kappa, &sh.gt_n);
            if (key > kappa && sg < kSMaxK) { sh.gt_key[sg] = key; sh.gt_col[sg] = col; }
            const bool eq = key == kappa && n_cut <= kSEqCap;
            const int se = wave_slot(eq, &sh.eq_n);
            if (eq && se < kSEqCap) sh.eq_col[se] = col;
        }
    } else {
        for_each_candidate([&](uint32_t key, int32_t col) {
            if (key > kappa) {
                const int slot = atomicAdd(&sh.gt_n, 1);
                if (slot < kSMaxK) { sh.gt_key[slot] = key; sh.gt_col[slot] = col; }
            } else if (key == kappa && n_cut <= kSEqCap) {
                const int slot = atomicAdd(&sh.eq_n, 1);
                if (slot < kSEqCap) sh.eq_col[slot] = col;
            }
        });
    }
    __syncthreads();
    const int n = count_gt;                                        // == sh.gt_n
    // sort by (key descending, column ascending): rank by counting, the n x n comparisons spread
    // over all threads (entry i = tid mod 256 against one part of the others each)
    if (tid < kSMaxK) sh.rank[tid] = 0;
    __syncthreads();
    {
        constexpr int kParts = kSThreads / kSMaxK;
        static_assert(kParts >= 1 && kParts * kSMaxK == kSThreads, "whole parts");
        const int i = tid & (kSMaxK - 1), part = tid / kSMaxK;
        if (i < n) {
            // four entries per LDS read, one 64-bit comparison per pair on (key, inverted column)
            const uint64_t mine = ((uint64_t)sh.gt_key[i] << 32) | (uint32_t)~sh.gt_col[i];
            const int per = ((n + kParts - 1) / kParts + 3) & ~3;
            const int e_begin = part * per;
            const int e_end = e_begin + per < n ? e_begin + per : n;
            int r = 0;
            for (int e = e_begin; e < e_end; e += 4) {
                const uint4 ok = *reinterpret_cast<const uint4*>(&sh.gt_key[e]);
                const int4 oc = *reinterpret_cast<const int4*>(&sh.gt_col[e]);
                r += (((uint64_t)ok.x << 32) | (uint32_t)~oc.x) > mine;
                r += e + 1 < e_end && (((uint64_t)ok.y << 32) | (uint32_t)~oc.y) > mine;
                r += e + 2 < e_end && (((uint64_t)ok.z << 32) | (uint32_t)~oc.z) > mine;
                r += e + 3 < e_end && (((uint64_t)ok.w << 32) | (uint32_t)~oc.w) > mine;
            }
            if (r != 0) atomicAdd(&sh.rank[i], r);
        }
    }
    __syncthreads();
    if (tid < n) {
        const int r = sh.rank[tid];
        sh.st_key[r] = sh.gt_key[tid];
        sh.st_col[r] = sh.gt_col[tid];
    }
    __syncthreads();

    // masses in rank order (fp64), cuts -----------------------------------------------------
    const uint32_t key1 = n > 0 ? sh.st_key[0] : kappa;           // the row's highest level
    const double z1 = (double)__uint_as_float(f32_of_key(key1));
    const double z_cut = (double)__uint_as_float(f32_of_key(kappa));
    if (tid < n) sh.st_M[tid] = exp(((double)__uint_as_float(f32_of_key(sh.st_key[tid])) - z1) * inv_tau);
    __syncthreads();
    if (tid < 64) {
        // wave 0: lane l holds sorted entries 4l .. 4l+3; inclusive prefix sums in rank order
        double w[4], loc = 0.0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int i = 4 * tid + j;
            w[j] = i < n ? sh.st_M[i] : 0.0;
            loc += w[j];
        }
        double run = wave_prefix_sum(loc) - loc;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int i = 4 * tid + j;
            run += w[j];
            if (i < n) sh.st_M[i] = run;
        }
    }
    __syncthreads();
    const double M_gt = n > 0 ? sh.st_M[n - 1] : 0.0;
    const double w_cut = exp((z_cut - z1) * inv_tau);
    const double M_k = M_gt + (double)n_cut * w_cut;              // mass of the top-k set
    // top-p on the renormalised top-k set: first level end whose cumulative mass reaches T
    if (tid == 0) sh.cut_index = kSMaxK;                           // default: everything down to the cut level
    __syncthreads();
    if (a.top_p < 1.0f) {
        const double Tm = (double)a.top_p * M_k;
        if (tid < n) {
            const bool level_end = tid == n - 1 || sh.st_key[tid + 1] != sh.st_key[tid];
            if (level_end && sh.st_M[tid] >= Tm) atomicMin(&sh.cut_index, tid);
        }
        __syncthreads();
    }
    const int cut_index = sh.cut_index;
    const bool cut_level_kept = cut_index == kSMaxK;
    const int kept_sorted = cut_level_kept ? n : cut_index + 1;    // sorted entries kept
    const int kept_C = cut_level_kept ? n + n_cut : kept_sorted;
    const double ln_M = wave == kSWaves - 1 ? log(cut_level_kept ? M_k : sh.st_M[cut_index]) : 0.0;      // the wave with the least of the race

    // race of the kept levels ------------------------------------------------------------------
    // score n_j w_j / E_j, E_j from Philox stream 3 at index = the level's stored pattern; fp32
    // scores as in the unrestricted sampler; ties go to the higher level = lower sorted index.
    const float z1f = __uint_as_float(f32_of_key(key1));
    auto level_score = [&](uint32_t key, int cnt) -> float {
        const uint32_t bits = f32_of_key(key);
        const uint32_t pat = T::pattern_of_bits(bits);
        uint32_t w4[4];
        philox4x32_10(pat >> 2, (uint32_t)grow, (uint32_t)(grow >> 32), 3u,
                      (uint32_t)a.seed, (uint32_t)(a.seed >> 32), w4);
        const int sel = pat & 3;
        const uint32_t word = sel == 0 ? w4[0] : sel == 1 ? w4[1] : sel == 2 ? w4[2] : w4[3];
        return (float)cnt * __builtin_amdgcn_exp2f((__uint_as_float(bits) - z1f) * c) * inv_exp_variate(word);
    };
    float my_q = -1.0f;
    int my_lvl = 0x7FFFFFFF;                                       // sorted index of the level's first entry; kSMaxK = cut level
    if (tid < kept_sorted) {
        const bool level_start = tid == 0 || sh.st_key[tid - 1] != sh.st_key[tid];
        if (level_start) {
            int cnt = 1;
            while (tid + cnt < n && sh.st_key[tid + cnt] == sh.st_key[tid]) ++cnt;
            my_q = level_score(sh.st_key[tid], cnt);
            my_lvl = tid;
        }
    } else if (tid == kSThreads - 1 && cut_level_kept) {
        my_q = level_score(kappa, n_cut);
        my_lvl = kSMaxK;
    }
    const Cand of_wave = wave_best(Cand{my_q, my_lvl});
    if (lane == 0) { sh.wave_q[wave] = of_wave.q; sh.wave_lvl[wave] = of_wave.idx; }
    __syncthreads();
    const Cand winner = row16_best(Cand{sh.wave_q[lane & (kSWaves - 1)], sh.wave_lvl[lane & (kSWaves - 1)]});
    const float best_q = winner.q;
    const int best_lvl = winner.idx;

    // the column inside the winning level ---------------------------------------------------------
    const uint64_t k23 = (uint64_t)sh.k23;
    int tok = 0;
    uint32_t tok_key = key1;
    if (best_q >= 0.0f && best_lvl < kSMaxK) {
        int cnt = 1;
        while (best_lvl + cnt < n && sh.st_key[best_lvl + cnt] == sh.st_key[best_lvl]) ++cnt;
        const int pos = (int)(((2u * k23 + 1u) * (uint64_t)cnt) >> 24);
        tok = sh.st_col[best_lvl + pos];                           // a level's entries are in column order
        tok_key = sh.st_key[best_lvl];
    } else if (best_q >= 0.0f) {
        const int pos = (int)(((2u * k23 + 1u) * (uint64_t)n_cut) >> 24);
        tok_key = kappa;
        if (n_cut <= kSEqCap) {
            // the pos-th smallest of the listed columns
            if (tid < n_cut) {
                const int32_t mc = sh.eq_col[tid];
                int rank = 0;
                for (int e = 0; e < n_cut; ++e) rank += sh.eq_col[e] < mc;
                if (rank == pos) sh.token = mc;
            }
            __syncthreads();
            tok = sh.token;
        } else {
            // a plateau: count the level's columns in column order; waves take contiguous runs of vectors
            const int64_t per_wave = (nvec + kSWaves - 1) / kSWaves;
            const int64_t v_begin = (int64_t)wave * per_wave < nvec ? (int64_t)wave * per_wave : nvec;
            const int64_t v_end = v_begin + per_wave < nvec ? v_begin + per_wave : nvec;
            auto mask_of = [&](int64_t v) -> uint32_t {
                const u32x4 x = rv[v];
                uint32_t m = 0;
#pragma unroll
                for (int e = 0; e < T::kElems; ++e)
                    m |= (uint32_t)(v * T::kElems + e < V && key_of_f32(T::elem_bits(x, e)) == kappa) << e;
                return m;
            };
            int hits = 0;
            for (int64_t v = v_begin + lane; v < v_end; v += 64) hits += __popc(mask_of(v));
#pragma unroll
            for (int d = 32; d > 0; d >>= 1) hits += __shfl_xor(hits, d, 64);
            if (lane == 0) sh.wave_hits[wave] = hits;
            __syncthreads();
            int before = 0;
            for (int w = 0; w < wave; ++w) before += sh.wave_hits[w];
            if (pos >= before && pos < before + hits) {            // uniform per wave: my run holds it
                int rem = pos - before;
                for (int64_t v0 = v_begin; v0 < v_end; v0 += 64) {
                    const int64_t v = v0 + lane;
                    const uint32_t m = v < v_end ? mask_of(v) : 0u;
                    const int cc = __popc(m);
                    int inc = cc;
#pragma unroll
                    for (int d = 1; d < 64; d <<= 1) {
                        const int o = __shfl_up(inc, d, 64);
                        if (lane >= d) inc += o;
                    }
                    const int sweep_total = __shfl(inc, 63, 64);
                    if (rem < sweep_total) {
                        if (rem >= inc - cc && rem < inc) {        // exactly one lane
                            int skip = rem - (inc - cc);
                            uint32_t mm = m;
                            while (skip-- > 0) mm &= mm - 1;       // drop the lowest set bits
                            sh.token = (int)(v * T::kElems + (__ffs(mm) - 1));
                        }
                        break;
                    }
                    rem -= sweep_total;
                }
            }
            __syncthreads();
            tok = sh.token;
        }
    }
    if (tid == kSThreads - 64) {
        if (tok < 0 || tok >= V) tok = 0;
        a.token_out[row] = tok;
        if (a.kept_out) a.kept_out[row] = kept_C;
        if (a.logp_out)
            a.logp_out[row] = best_q >= 0.0f
                ? (float)(((double)__uint_as_float(f32_of_key(tok_key)) - z1) * inv_tau - ln_M)
                : __builtin_nanf("");
    }
}

}  // namespace

bool sample_select_serves(int32_t top_k) { return top_k >= 1 && top_k <= kSMaxK; }

hipError_t launch_sample_select(const void* logits, bool is_bf16, int64_t rows, int64_t V, int64_t row_stride,
                                const float* tau_rows, float tau_scalar, int32_t top_k, float top_p,
                                uint64_t seed, uint64_t row_base, int32_t* token_out,
                                float* logp_out, int32_t* kept_out, hipStream_t stream)
{
    if (rows == 0) return hipSuccess;
    SelArgs a;
    a.logits = logits; a.rows = rows; a.V = V; a.row_stride = row_stride;
    a.tau_rows = tau_rows; a.tau_scalar = tau_scalar;
    a.top_k = top_k; a.top_p = top_p;
    a.seed = seed; a.row_base = row_base;
    a.token_out = token_out; a.logp_out = logp_out; a.kept_out = kept_out;
    const bool few = rows <= compute_units();
    if (is_bf16) {
        if (few) hipLaunchKernelGGL((sample_select_kernel<SelBf16, 1024>), dim3((unsigned)rows), dim3(1024), 0, stream, a);
        else hipLaunchKernelGGL((sample_select_kernel<SelBf16, 512>), dim3((unsigned)rows), dim3(512), 0, stream, a);
    } else {
        if (few) hipLaunchKernelGGL((sample_select_kernel<SelF32, 1024>), dim3((unsigned)rows), dim3(1024), 0, stream, a);
        else hipLaunchKernelGGL((sample_select_kernel<SelF32, 512>), dim3((unsigned)rows), dim3(512), 0, stream, a);
    }
    return hipGetLastError();
}

}  // namespace e3
