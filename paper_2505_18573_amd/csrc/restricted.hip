// Restricted (top-k / top-p) sampling of bf16 logit rows for gfx950.
//
// Paper: arXiv 2505.18573 samples its rollouts unrestricted at temperature tau
// (Section 5.1); rollout engines usually offer both truncations, so the definition is
// the library's own and is stated in include/e3.h: columns that store one bit pattern
// form a LEVEL, levels are ranked by value, the cuts are taken on cumulative level
// counts (top-k) and cumulative level masses (top-p), and the draw is a Gumbel-max
// over the kept levels followed by a uniform choice among the winning level's columns.
//
// bf16 has only 65,536 bit patterns, so the whole value distribution of a row is a count
// histogram.  One workgroup owns one row:
//   1. stream the row once, counting with LDS atomics;
//   2. every thread owns a run of consecutive levels of one binade, i.e. equally spaced
//      values whose weights exp((z - z_1)/tau) form a geometric sequence: two
//      exponentials and a product per level give all level masses in fp64; a workgroup
//      scan yields the cumulative counts C_j and masses M_j in rank order;
//   3. the cuts are located by the thread whose levels contain them, the kept levels
//      race for the draw (n_j w_j / E_j, fp32 like the unrestricted sampler), and the
//      pos-th column of the winning level is looked up in the row.
// Counts are integers; masses and the cuts are fp64.
//
// THE NEAR WINDOW (every ordinary row).  The values a row really holds span few binades: 31.5 binades of
// both signs, 8064 levels, are counted in 64 KiB of LDS - those up to [256, 512), or up to one above the
// magnitude of the largest logit among the first vectors read, whichever is higher.  64 KiB instead of
// the 128 KiB all patterns need is what lets two rows share a compute unit, so that one row's short
// dependent phases overlap the other's stream.  Each level has four 16-bit counters, one
// per quarter of the row (the quarter is uniform per step of the stream, so it costs nothing), and
// the final look-up reads only the quarter that holds the column.  What lies outside the
// window is kept exactly too: zeros are counted apart, up to 62 nearer to zero than the window are
// listed with their columns (the MIDDLE items, ranked between the two signs), and values
// below the window (masked columns) are counted when they are too far down to weigh anything; a
// count cut among them keeps all of them if they are one value.
//
// What bounds it.  The counting: an LDS atomic on 64 random counters takes 7.7 cycles (4 without a bank
// conflict), 7.6 us for the 151,936 columns of a row alone on its compute unit, and five vector
// instructions go with it; two rows together sit between that, the issue of those instructions and HBM.
// Then five short phases per row (levels and scan 2.0 us, cuts 1.2, race 0.9, look-up 2.2 to 3), chains of
// LDS, barriers and dependent instructions that the last rows of a launch have nothing to overlap with.
// Hence workgroups of eight waves (per-wave work of the phases is done half as often as with sixteen:
// 100 rows x 1000 columns 14.6 us with sixteen waves and 64 registers each, 9.8 now), two sets of requests in
// flight, and nothing in the stream but the count: spare words for what lies outside, one check per set.
// Sixteen waves still stream a single row faster: with at most one row per compute unit they win from
// about 114,688 columns on (eight / sixteen waves in us: 100 rows x 70,000 15.3 / 15.5, x 100,000 17.5 / 17.6, x 130,000 20.3 /
// 19.5, x 400,000 45.3 / 39.4; 256 rows x 40,000 13.6 / 15.1, x 100,000 19.0 / 19.4, x 130,000 21.6 / 21.5).
// Captured launches, top-p 0.9, sixteen waves with a burst of four requests / now: 8 x 151,936 23.0 /
// 18.3 us, 256 rows 26.2 / 22.2, 512 rows 43.2 / 37.2 (4.2 TB/s), 1024 rows 82.6 / 72.1; 512 x 32,000 26.7 / 15.9,
// 300 x 70,000 30.8 / 21.1, 512 x 5000 22.6 / 11.5.
//
// FEW ROWS, given a workspace.  A row alone on its compute unit is bound by that unit's LDS while the others idle.
// Such rows are cut into eight slices, each counted by a workgroup of its own in the window that 64 vectors spread over the row
// choose for all of them; 16 KiB of counters and some notes per slice go to memory (5 us), and the second launch
// adds the slices up (a quarter is two of them), runs the phases, and looks the column up in one slice (10 us).
// Where that sample holds neither large values nor negative ones of ordinary size, the window is lowered to the values it
// does hold, so that a row of small ones needs no list; if a slice then meets others, the second launch counts the
// row anew (8 x 151,936 clamped to at most 0: 268 us when the window followed the largest value alone, and the
// negative columns lay below it, 23 so; 3e-4 x ordinary with 30 columns at -30: 150 and 24).
// 8 x 151,936, top-p 0.9: 18.3 us whole, 14.2 cut; with 100 columns allowed and -1e4 elsewhere 57 and 23 us.
//
// A row with values above the window, or with more small ones than the list holds, is counted once
// more in a window raised to the former or lowered for the latter; its waves give the first count up as
// soon as they see it (151,936 columns, 8 / 512 rows: a logit of 9000 at the end of the row 37 / 46 us, all logits
// around -2000, seen by the first vectors, 34 / 61 us, all below 1e-3 38 / 58 us).
//
// THE WIDE ROWS.  Everything else - a second window that fails too, a wrapped counter (recognised
// because the counts no longer add up to the row's width), a count cut among several levels below the
// window, columns below it that still weigh something (a mask of -1e4 at tau above 178) - is redone
// over all patterns with 32-bit counters, in four windows of 16,384 patterns in rank order, one
// sweep each; a cut or the race needs its window swept again unless it was the last.  Slow (up
// to ten sweeps), exact, rare: ordinary logits with 500 columns of 2^-24 to 2^-60 among them 86 / 148 us at 8 /
// 512 rows, the first half of 400,000 columns equal 345 us at 8 rows.  Its code is inlined
// although few rows run it: as a function of its own the calling convention cost every row scratch
// memory (8 ordinary rows 25 -> 31 us, 512 rows 45 -> 63 us).
#include "vocab_common.h"
#include "vocab_pass.h"
#include "wave_scan.h"

namespace e3 {
namespace {

constexpr int kBinades = 32;                    // of each sign in the near window
constexpr int kHalf = kBinades * 128;           // its words of one sign
constexpr int kTopExp = 135;                    // exponent field of the lowest top binade, [256, 512)
constexpr int kTopEnd = (kTopExp + 1) << 7;     // the first magnitude above it
constexpr int kQuarters = 4;
constexpr int kTrash = 64;                      // spare words, one per lane
constexpr int kLevels = kHalf - kTrash;         // levels of one sign that are counted
constexpr int kArray = 2 * kHalf;               // words of two quarters' counters
constexpr int kWideBins = 16384;                // patterns in one of the four wide windows
constexpr int kWideWindows = 4;
constexpr int kMidList = 62;                    // listed small values; with the two zeros one item per lane
// Stream steps of one set of requests, two sets being in flight: 512 x 151,936 37.7, 38.8 and 39.7 us with 2, 3 and 4
// (the first values arrive later the more are asked for), 8 x 151,936 20.0, 19.9 and 20.1.
constexpr int kSet = 2;
static_assert(kArray * 2 >= kWideBins, "the wide window fits the same memory");

// Rank key of a pattern: ascending in value, -0 just below +0.
__device__ __forceinline__ int key_of_pattern(int p) { return p < 0x8000 ? p + 0x8000 : 0xFFFF - p; }
__device__ __forceinline__ int pattern_of_key(int key) { return key >= 0x8000 ? key - 0x8000 : 0xFFFF - key; }
__device__ __forceinline__ float value_of_pattern(int p) { return __uint_as_float((uint32_t)p << 16); }

struct RestrictedArgs {
    const uint16_t* logits;
    int64_t rows, V, row_stride;
    const float* tau_rows;
    float tau_scalar;
    int32_t top_k;
    float top_p;
    uint64_t seed, row_base;
    int32_t* token_out;
    float* logp_out;
    int32_t* kept_out;
    // rows cut into slices (few rows): how many, their counters and what they found outside the window
    int32_t nslices;
    uint16_t* slice_counts;         // [rows][nslices][2 kHalf]
    struct SliceNotes* slice_notes; // [rows][nslices]
};

// What a slice of a row passes on besides its counters.  The window is the same for all slices of a row.
struct alignas(16) SliceNotes {
    int zeros[2];                   // +0, -0
    int list_n, n_below, n_not_finite, below_lo, below_hi;
    int above_hi;                   // not 0: the largest of the columns above the window (of those seen, the count stops then)
    int base;
    float first_top;
    int list_key[kMidList], list_col[kMidList];
};

// A row's sampling by one workgroup of kRThreads threads.
template <int kRThreads>
struct Sampler {
static constexpr int kRWaves = kRThreads / 64;
static constexpr int kOwnN = 2 * kHalf / kRThreads;    // near window: a thread's levels
static constexpr int kOwnW = kWideBins / kRThreads;
static constexpr int kWideSet = 2048 / kRThreads;      // wide rows: stream steps of one set of requests
// Stream steps looked up at a time: one block is enough for a quarter of up to 163,840 columns.
static constexpr int kBlock = 5120 / kRThreads;
static constexpr int kShortBlock = 3;
static_assert(kOwnN * kRThreads == 2 * kHalf && 128 % kOwnN == 0 && 128 % kOwnW == 0, "a thread's levels share a binade");

struct Shared {
    float wave_top[kRWaves];
    double wave_M[kRWaves];
    int wave_C[kRWaves];
    Cand best[kRWaves];
    float sample_max[kRWaves];
    float sample_mag;               // slices: the largest magnitude in the sample that the ordinary window holds
    int zeros[2][kQuarters];        // +0, -0 by quarter
    int list_n, n_below, n_not_finite, n_above;
    int below_lo, below_hi, above_hi;            // magnitude bits of the columns below the window (both ends) and above it
    int fails;                      // not 0: columns above the window, or more small ones than the list holds
    int list_key[64], list_col[64]; // small values as they come
    int mid_key[64], mid_cnt[64], mid_col[64];   // the middle items in rank order
    int mid_C[64];                  // inclusive prefixes inside the middle
    double mid_M[64];
    int cut_key[kRWaves + 1], cut_C[kRWaves + 1];      // what each wave (and the middle) offers as the cut
    double cut_M[kRWaves + 1];
    int tot[kBlock * kRWaves];
    int C_above[kWideWindows + 1];  // wide rows: count and mass above each window
    double M_above[kWideWindows + 1];
};

// The row as 16-byte vectors, kRThreads of them per step.  The last vector may reach past the row's
// columns (inside the row pitch, whose 16-byte multiple the interface demands): what it holds
// there, and vectors past the row, read as patterns that are not numbers.
struct Row {
    const u32x4* p;
    int nvec, last;       // vectors; columns in the last one, 1 .. 8
    int complete;         // vectors of eight columns
    int steps, whole;     // steps, and how many of them hold nothing but complete vectors
    // vectors [v0, v1) of the row
    __device__ __forceinline__ Row part(int v0, int v1) const
    {
        Row q;
        q.p = p + v0;
        q.nvec = v1 - v0;
        q.last = v1 == nvec ? last : 8;
        q.complete = q.nvec - (q.last < 8);
        q.steps = (q.nvec + kRThreads - 1) / kRThreads;
        q.whole = q.complete / kRThreads;
        return q;
    }
    // slice s of n
    __device__ __forceinline__ int slice_begin(int s, int n) const { return (int)((int64_t)nvec * s / n); }
    // vector v without what is not the row's
    __device__ __forceinline__ u32x4 counted(const u32x4& x, int v) const
    {
        constexpr uint32_t kNone = 0xFFC0FFC0u;
        const int n = v < nvec - 1 ? 8 : v == nvec - 1 ? last : 0;
        auto fill = [&](uint32_t word, int first) -> uint32_t {
            return n <= first ? kNone : n == first + 1 ? (word & 0xFFFFu) | (kNone & 0xFFFF0000u) : word;
        };
        return u32x4{fill(x.x, 0), fill(x.y, 2), fill(x.z, 4), fill(x.w, 6)};
    }
    // kN steps from `step` on, requested together and without a branch (where two sides of one meet, the
    // compiler waits for the loads of both): past the row they repeat its last vector, for `counted` to drop
    template <int kN>
    __device__ __forceinline__ void request_ahead(u32x4 x[kN], int step, int tid) const
    {
#pragma unroll
        for (int u = 0; u < kN; ++u) {
            const int v = tid + (step + u) * kRThreads;
            x[u] = p[v < nvec ? v : nvec - 1];
        }
    }
};

static __device__ __forceinline__ Row whole_row(const RestrictedArgs& a, int64_t r)
{
    Row row;
    row.p = reinterpret_cast<const u32x4*>(a.logits + r * a.row_stride);
    row.nvec = (int)((a.V + 7) >> 3);
    row.last = (int)(a.V - ((int64_t)(row.nvec - 1) << 3));
    row.steps = (row.nvec + kRThreads - 1) / kRThreads;
    row.complete = (int)(a.V >> 3);
    row.whole = row.complete / kRThreads;
    return row;
}

template <typename F>
static __device__ __forceinline__ void for_each_pattern(const u32x4& v, F&& f)
{
    f(v.x & 0xFFFFu, 0); f(v.x >> 16, 1); f(v.y & 0xFFFFu, 2); f(v.y >> 16, 3);
    f(v.z & 0xFFFFu, 4); f(v.z >> 16, 5); f(v.w & 0xFFFFu, 6); f(v.w >> 16, 7);
}

// A thread's levels after the scan: levels of one binade in falling rank order, `top` the first
// with columns (weight w_top, at most 1), each later one `r` times the weight of the one before.
struct View {
    int top;
    double w_top, r;
    int Cl, Cx;           // my count; count of all higher levels
    double Ml, Mx;        // the same for mass
};

// The weight after level j's: levels before `top` have no columns and keep w_top (their own weight
// may lie beyond fp64 when the thread holds levels above the row's highest).
static __device__ __forceinline__ double next_weight(const View& vw, double w, int j) { return j < vw.top ? w : w * vw.r; }

// Weights and mass of a thread's levels: cnt(j) columns on level j, z_top the value of level `top`,
// e the binade's exponent field.
template <int kOwn, int kUnroll, typename Cnt>
static __device__ __forceinline__ void own_mass(View& vw, int e, float z_top, double z1, double inv_tau, Cnt&& cnt)
{
    vw.w_top = 0.0; vw.r = 0.0; vw.Ml = 0.0;
    if (vw.Cl > 0) {
        vw.w_top = exp(((double)z_top - z1) * inv_tau);
        vw.r = exp(-ldexp(1.0, (e ? e : 1) - 134) * inv_tau);
        // from the lowest level up, in units of level `top`'s weight: levels above it have no columns and leave the sum alone
        double m = 0.0;
#pragma unroll kUnroll
        for (int j = kOwn - 1; j >= 0; --j) {
            const uint32_t n = (uint32_t)cnt(j);
            const double up = fma(m, vw.r, (double)n);
            m = j >= vw.top ? up : m;
        }
        vw.Ml = m * vw.w_top;
    }
}

// Inclusive prefixes over the waves, one wave per lane of the first sixteen: lanes kRWaves - 1 to 15 hold the totals, lanes behind them nothing.
struct Waves { int C; double M; };

// Exclusive scan of counts and masses in thread order = rank order; threads from `mid_at` on
// also have the middle's totals before them, which one wave has left in LDS.  Returns the scanned levels' prefixes over the waves.
static __device__ __forceinline__ Waves scan_view(View& vw, int carry_C, double carry_M, int mid_at, Shared& sh, int tid)
{
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int Ci = 0;
    double Mi = 0.0;
    if (__any(vw.Cl > 0)) wave_prefix_sum2(vw.Cl, vw.Ml, Ci, Mi);
    if (lane == 63) { sh.wave_C[wave] = Ci; sh.wave_M[wave] = Mi; }
    __syncthreads();
    Waves all;
    row16_prefix_sum2(lane < kRWaves ? sh.wave_C[lane & (kRWaves - 1)] : 0, lane < kRWaves ? sh.wave_M[lane & (kRWaves - 1)] : 0.0, all.C, all.M);
    int Cb = carry_C;
    double Mb = carry_M;
    if (wave > 0) { Cb += __builtin_amdgcn_readlane(all.C, wave - 1); Mb += read_lane(all.M, wave - 1); }
    if (tid >= mid_at) { Cb += sh.mid_C[63]; Mb += sh.mid_M[63]; }
    vw.Cx = Cb + Ci - vw.Cl;
    vw.Mx = Mb + (Mi - vw.Ml);
    return all;
}

// Cut search among one thread's levels: the level whose cumulative count reaches k.
struct Cut { int j, C; double M; };       // level j of the thread; count and mass down to it

template <int kOwn, int kUnroll, typename Cnt>
static __device__ __forceinline__ Cut own_count_cut(const View& vw, int k, Cnt&& cnt)
{
    Cut cut{kOwn - 1, vw.Cx, vw.Mx};
    double w = vw.w_top;
    bool done = false;
#pragma unroll kUnroll
    for (int j = 0; j < kOwn; ++j) {
        const int n = (int)cnt(j);
        if (!done) {
            cut.j = j; cut.C += n; cut.M = fma((double)n, w, cut.M);
            done = cut.C >= k;
        }
        w = next_weight(vw, w, j);
    }
    return cut;
}
// The mass cut of the workgroup: the owner is the first thread in rank order whose inclusive prefix
// reaches T (the scan's prefixes may disagree in the last bit, so only threads with columns count),
// the cut its first populated level whose cumulative mass reaches T, or the lowest populated one
// if rounding lets none reach it.  Every wave's first such thread is looked through by the wave, one level
// per lane (count_at(rank) from LDS), and the result offered; the lowest wave's offer is taken.
template <int kOwn, typename CountAt, typename KeyAt>
static __device__ __forceinline__ void offer_mass_cut(const View& vw, double T, CountAt&& count_at, KeyAt&& key_at, Shared& sh, int tid)
{
    static_assert(kOwn <= 64, "a lane per level");
    const int lane = tid & 63, wave = tid >> 6;
    const unsigned long long reach = __ballot(vw.Cl > 0 && vw.Mx + vw.Ml >= T);
    // (a wave with clearly more than T above it cannot be the lowest)
    if (reach == 0ull || read_lane(vw.Mx, 0) > T * (1.0 + 1e-9)) {
        if (lane == 0) sh.cut_key[wave] = -1;
        return;
    }
    const int owner = (int)__builtin_ctzll(reach);
    const int rank = kOwn * (wave * 64 + owner) + lane;
    const int n = lane < kOwn ? (int)count_at(rank) : 0;
    const int e = lane - __builtin_amdgcn_readlane(vw.top, owner);        // lanes before the owner's top level have n == 0
    double w = read_lane(vw.w_top, owner), r = read_lane(vw.r, owner);
#pragma unroll
    for (int bit = 1; bit < kOwn; bit <<= 1) {
        if (e > 0 && (e & bit) != 0) w *= r;
        r *= r;
    }
    const int C = __builtin_amdgcn_readlane(vw.Cx, owner) + wave_prefix_sum(n);
    const double M = read_lane(vw.Mx, owner) + wave_prefix_sum(n != 0 ? (double)n * w : 0.0);
    const unsigned long long have = __ballot(n != 0), enough = __ballot(n != 0 && M >= T);
    const int at = enough != 0ull ? (int)__builtin_ctzll(enough) : 63 - (int)__builtin_clzll(have);
    if (lane == at) { sh.cut_key[wave] = key_at(rank); sh.cut_C[wave] = C; sh.cut_M[wave] = M; }
}
// The first wave with an offer, or kRWaves.
static __device__ __forceinline__ int first_offer(const Shared& sh, int lane)
{
    const unsigned long long have = __ballot(lane < kRWaves && sh.cut_key[lane & (kRWaves - 1)] >= 0);
    return have != 0ull ? (int)__builtin_ctzll(have) : kRWaves;
}

// A contestant of the race: score n w / E and a label that is lower for a higher level (ties go
// to the higher level, as Cand's go to the lower label).
static __device__ __forceinline__ Cand contestant(float q, int key) { return Cand{q, 0xFFFF - key}; }
static __device__ __forceinline__ int key_of(const Cand& c) { return 0xFFFF - c.idx; }

// Score of the level with pattern p and n columns: n 2^{(z - z_1) c} / E, E = -ln u from Philox
// stream 3 at index = the pattern.  fp32, as in the unrestricted sampler; decisions closer than
// fp32 resolves are the near-ties the parity rule exempts.
static __device__ __forceinline__ float level_score(int p, int n, float z1f, float c, uint64_t seed, uint64_t grow)
{
    uint32_t w4[4];
    philox4x32_10((uint32_t)p >> 2, (uint32_t)grow, (uint32_t)(grow >> 32), 3u, (uint32_t)seed, (uint32_t)(seed >> 32), w4);
    const int sel = p & 3;
    const uint32_t word = sel == 0 ? w4[0] : sel == 1 ? w4[1] : sel == 2 ? w4[2] : w4[3];
    return (float)n * __builtin_amdgcn_exp2f((value_of_pattern(p) - z1f) * c) * inv_exp_variate(word);
}

// The workgroup's best contestant.
static __device__ __forceinline__ Cand reduce_best(Cand b, Shared& sh, int tid)
{
    const int lane = tid & 63;
    b = wave_best(b);
    if (lane == 0) sh.best[tid >> 6] = b;
    __syncthreads();
    static_assert(kRWaves <= 16, "one lane of a sixteen-lane row per wave");
    return row16_best(sh.best[lane & (kRWaves - 1)]);
}

typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
typedef int16_t s16x2 __attribute__((ext_vector_type(2)));
static __device__ __forceinline__ u16x2 halves(uint32_t w) { return __builtin_bit_cast(u16x2, w); }
static __device__ __forceinline__ s16x2 signed_halves(uint32_t w) { return __builtin_bit_cast(s16x2, w); }

// Stores the rem-th column (0-based, in column order) that holds pattern `pat` within stream steps
// [i0, i1): kBlock steps are requested at once; a (step, wave) holds 512 consecutive columns, so the
// waves' counts per step, in that order, say where the column is, and the wave that holds it
// finds the lane, which stores it (`row` starts at column col0).  0 if there are not that many.  Most (step, wave) hold no such column.
template <int kBlock>
static __device__ __forceinline__ void locate(const Row& row, int col0, int i0, int i1, uint32_t pat, int rem, int32_t* token,
                                       Shared& sh, int tid)
{
    const int lane = tid & 63, wave = tid >> 6;
    const u16x2 p2 = halves(pat | pat << 16);
#pragma unroll 1
    for (int ib = i0; ib < i1; ib += kBlock) {
        u32x4 x[kBlock];
        row.template request_ahead<kBlock>(x, ib, tid);
        int totals = 0;                                           // lane u: the wave's columns of step u
        uint32_t found[kBlock];                                   // my columns (bits 0..7) and how many my wave has up to me
#pragma unroll
        for (int u = 0; u < kBlock; ++u) {
            const u16x2 d = __builtin_elementwise_min(
                __builtin_elementwise_min(halves(x[u].x) ^ p2, halves(x[u].y) ^ p2),
                __builtin_elementwise_min(halves(x[u].z) ^ p2, halves(x[u].w) ^ p2));
            const int step = ib + u;
            found[u] = 0u;
            int total = 0;
            if (__any(d.x == 0 || d.y == 0) && step < i1) {       // uniform
                const int v = tid + step * kRThreads;
                uint32_t m = 0u;
                for_each_pattern(x[u], [&](uint32_t p, int j) { m |= (uint32_t)(p == pat) << j; });
                if (step >= row.whole) m = v < row.nvec - 1 ? m : v == row.nvec - 1 ? m & (0xFFu >> (8 - row.last)) : 0u;
                const int upto = wave_prefix_sum((int)__popc(m));
                found[u] = (uint32_t)upto << 8 | m;
                total = __builtin_amdgcn_readlane(upto, 63);
            }
            totals = lane == u ? total : totals;
        }
        if (lane < kBlock) sh.tot[lane * kRWaves + wave] = totals;
        __syncthreads();
        // every wave finds the (step, wave) that holds the column: two consecutive totals per lane
        static_assert(kBlock * kRWaves <= 128 && kBlock * kRWaves % 2 == 0, "two totals per lane");
        const bool some = 2 * lane < kBlock * kRWaves;
        const int t0 = some ? sh.tot[2 * lane] : 0, t1 = some ? sh.tot[2 * lane + 1] : 0;
        const int upto = wave_prefix_sum(t0 + t1);
        const unsigned long long past = __ballot(upto > rem);
        if (past != 0ull) {                                       // uniform over the workgroup
            const int l = (int)__builtin_ctzll(past);
            int before = __builtin_amdgcn_readlane(upto - t0 - t1, l);
            const int first = __builtin_amdgcn_readlane(t0, l);
            int at = 2 * l;
            if (before + first <= rem) { before += first; ++at; }
            if (at % kRWaves == wave) {
                const int step = at / kRWaves, want = rem - before;
                uint32_t mine = found[0];
#pragma unroll
                for (int u = 1; u < kBlock; ++u) mine = u == step ? found[u] : mine;
                uint32_t m = mine & 0xFFu;
                const int skip = want - ((int)(mine >> 8) - __popc(m));
                if (skip >= 0 && skip < __popc(m)) {              // exactly one lane
                    for (int i = 0; i < skip; ++i) m &= m - 1;
                    *token = col0 + (tid + (ib + step) * kRThreads) * 8 + (__ffs(m) - 1);
                }
            }
            return;
        }
        rem -= __builtin_amdgcn_readlane(upto, 63);
        __syncthreads();                                          // the totals are reused
    }
    if (tid == 0) *token = 0;                                     // only with weights that are no numbers
}

// The row's other outputs, by one thread; ln_M: the kept levels' mass relative to the weight of z_ref.
static __device__ __forceinline__ void store_row(const RestrictedArgs& a, int64_t r, int kept_C, bool drawn, int pattern,
                                          double z_ref, double ln_M, double inv_tau)
{
    if (a.kept_out) a.kept_out[r] = kept_C;
    if (a.logp_out)
        a.logp_out[r] = drawn ? (float)(((double)value_of_pattern(pattern) - z_ref) * inv_tau - ln_M)
                              : __builtin_nanf("");
    if (!drawn) a.token_out[r] = 0;
}

// ---------------------------------------------------------------------------
// The wide rows: four windows of 16,384 patterns in rank order, 32-bit counters.
// ---------------------------------------------------------------------------
struct WideWindow {
    int w;                                                        // 0: [2, inf), 1: [+0, 2), 2: (-2, -0], 3: (-inf, -2]
    __device__ __forceinline__ uint32_t quadrant() const { return w == 0 ? 1u : w == 1 ? 0u : (uint32_t)w; }
    __device__ __forceinline__ int pattern(int rank) const        // rank 0 = highest value
    {
        return (int)(quadrant() << 14) + (w < 2 ? kWideBins - 1 - rank : rank);
    }
};

// A pattern's counter in its window: neighbouring threads' runs of kOwnW start in different banks.
static __device__ __forceinline__ uint32_t wide_place(uint32_t p) { return (p & 0x3FFFu) ^ (p / kOwnW & 31u); }

// `resident` is the window that the counters hold already (-1: none).  Two sets of requests in flight and two patterns
// at a time, as in near_count: relative to the window's quadrant its own patterns have no high bits, and a minimum sends all
// others to the lane's spare word (8 x 151,936, top-p 0.9, with 500 small columns: 137 us when eight requests were waited for
// and then counted, 118 so).
static __device__ __forceinline__ void wide_count(const Row& row, WideWindow win, int& resident, uint32_t* hist, int tid)
{
    __syncthreads();
    if (win.w == resident) return;                                // uniform
    resident = win.w;
    u32x4 x[kWideSet], y[kWideSet];
    row.template request_ahead<kWideSet>(x, 0, tid);
    row.template request_ahead<kWideSet>(y, kWideSet, tid);
    for (int i = tid; i < (kWideBins + kTrash) / 4; i += kRThreads) reinterpret_cast<uint4*>(hist)[i] = uint4{0u, 0u, 0u, 0u};
    // orders LDS only: __syncthreads() would wait for the loads in flight as well
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    const uint32_t quad = win.quadrant() * 0x40004000u;
    const uint16_t spare = (uint16_t)(kWideBins + (tid & 63));
    const u16x2 spare_v = {spare, spare};
    static_assert(kWideBins == 0x4000 && kTrash == 64, "what exceeds a place is a spare word or above all of them");
    auto add2 = [&](uint32_t word) {
        const uint32_t t = word ^ quad;
        const uint32_t at = __builtin_bit_cast(uint32_t, __builtin_elementwise_min(halves(t ^ (t / kOwnW & 0x001F001Fu)), spare_v));
        atomicAdd(&hist[at & 0xFFFFu], 1u);
        atomicAdd(&hist[at >> 16], 1u);
    };
    auto count = [&](const u32x4 (&x)[kWideSet], int i0) {
#pragma unroll
        for (int u = 0; u < kWideSet; ++u) {
            const int step = i0 + u;
            if (step >= row.steps) break;                         // uniform
            const u32x4 v = step < row.whole ? x[u] : row.counted(x[u], tid + step * kRThreads);
            add2(v.x); add2(v.y); add2(v.z); add2(v.w);
        }
    };
#pragma unroll 1
    for (int i0 = 0; i0 < row.steps; i0 += 2 * kWideSet) {
        count(x, i0);
        row.template request_ahead<kWideSet>(x, i0 + 2 * kWideSet, tid);
        count(y, i0 + kWideSet);
        row.template request_ahead<kWideSet>(y, i0 + 3 * kWideSet, tid);
    }
    __syncthreads();
}

static __device__ __forceinline__ void wide_row(const Row& row, const RestrictedArgs& a, int64_t r, double inv_tau, float c,
                                         uint64_t grow, uint32_t k23, uint32_t* hist, Shared& sh, int tid)
{
    const int lane = tid & 63, wave = tid >> 6;
    const bool k_on = a.top_k >= 1 && (int64_t)a.top_k < a.V, p_on = a.top_p < 1.0f;
    auto count_of = [&](WideWindow win, int rank) -> uint32_t {
        const int p = win.pattern(rank);
        return ((p >> 7) & 0xFF) == 0xFF ? 0u : hist[wide_place((uint32_t)p)];
    };
    int resident = -1;
    double z1 = 0.0;
    bool have_z1 = false;
    // counts the window and scans it; (C, M) = what lies above it on entry, with it on return
    auto scan = [&](WideWindow win, View& vw, int& C, double& M) {
        wide_count(row, win, resident, hist, tid);
        // My levels, read once: one binade, and one aligned run of words up to the exchange in wide_place.  (Each one's place
        // and exponent worked out anew, for the count and for the mass, in a loop of eight: the 118 us above, 86 so; one copy of
        // this code for all sweeps instead of three: 5 us more.)
        uint32_t cnt[kOwnW];
        const int p0 = win.pattern(kOwnW * tid), run = p0 & 0x3FFF & ~(kOwnW - 1);
        const int exchange = run / kOwnW % 32 ^ (win.w < 2 ? kOwnW - 1 : 0);
        const bool numbers = ((p0 >> 7) & 0xFF) != 0xFF;
#pragma unroll
        for (int j = 0; j < kOwnW; ++j) cnt[j] = hist[run ^ exchange ^ j];
        vw.Cl = 0; vw.top = kOwnW;
#pragma unroll
        for (int j = kOwnW - 1; j >= 0; --j) {
            if (!numbers) cnt[j] = 0u;
            vw.Cl += (int)cnt[j];
            if (cnt[j] != 0u) vw.top = j;
        }
        const int p_top = win.pattern(kOwnW * tid + (vw.Cl > 0 ? vw.top : 0));
        if (!have_z1) {
            const float t = wave_max(vw.Cl > 0 ? (float)key_of_pattern(p_top) : -1.0f);
            if (lane == 0) sh.wave_top[wave] = t;
            __syncthreads();
            const float best = row16_max(sh.wave_top[lane & (kRWaves - 1)]);
            if (best >= 0.0f) { have_z1 = true; z1 = (double)value_of_pattern(pattern_of_key((int)best)); }
        }
        own_mass<kOwnW, kOwnW>(vw, (p_top >> 7) & 0xFF, value_of_pattern(p_top), z1, inv_tau, [&](int j) { return cnt[j]; });
        const Waves all = scan_view(vw, C, M, kRThreads, sh, tid);
        C += __builtin_amdgcn_readlane(all.C, kRWaves - 1); M += read_lane(all.M, kRWaves - 1);
    };
    int C_all = 0;
    double M_all = 0.0;
#pragma unroll 1
    for (int w = 0; w < kWideWindows; ++w) {
        if (tid == 0) { sh.C_above[w] = C_all; sh.M_above[w] = M_all; }
        View vw;
        scan(WideWindow{w}, vw, C_all, M_all);
    }
    if (tid == 0) { sh.C_above[kWideWindows] = C_all; sh.M_above[kWideWindows] = M_all; }
    __syncthreads();
    if (!have_z1) {                                               // no finite logit
        if (tid == 0) store_row(a, r, 0, false, 0, 0.0, 0.0, inv_tau);
        return;
    }
    int cut_key = 0, kept_C = C_all;
    double kept_M = M_all;
    // one sweep of the window that holds a cut, then the owner's search
    if (k_on && kept_C >= a.top_k) {
#pragma unroll 1
        for (int w = 0; w < kWideWindows; ++w) {
            if (sh.C_above[w] < a.top_k && sh.C_above[w + 1] >= a.top_k) {
                const WideWindow win{w};
                View vw;
                int C = sh.C_above[w];
                double M = sh.M_above[w];
                scan(win, vw, C, M);
                if (vw.Cx < a.top_k && vw.Cx + vw.Cl >= a.top_k) {          // one thread
                    const Cut cut = own_count_cut<kOwnW, 1>(vw, a.top_k, [&](int j) { return count_of(win, kOwnW * tid + j); });
                    sh.cut_key[0] = key_of_pattern(win.pattern(kOwnW * tid + cut.j)); sh.cut_C[0] = cut.C; sh.cut_M[0] = cut.M;
                }
                __syncthreads();
            }
        }
        cut_key = sh.cut_key[0]; kept_C = sh.cut_C[0]; kept_M = sh.cut_M[0];
        __syncthreads();
    }
    if (p_on) {
        const double T = (double)a.top_p * kept_M;
        bool looked = false;
#pragma unroll 1
        for (int w = 0; w < kWideWindows; ++w) {
            if (!looked && sh.C_above[w + 1] > sh.C_above[w] && sh.M_above[w + 1] >= T) {
                looked = true;
                const WideWindow win{w};
                View vw;
                int C = sh.C_above[w];
                double M = sh.M_above[w];
                scan(win, vw, C, M);
                offer_mass_cut<kOwnW>(vw, T, [&](int rank) { return count_of(win, rank); },
                                      [&](int rank) { return key_of_pattern(win.pattern(rank)); }, sh, tid);
                __syncthreads();
                const int w1 = first_offer(sh, lane);
                if (w1 < kRWaves && sh.cut_key[w1] > cut_key) { cut_key = sh.cut_key[w1]; kept_C = sh.cut_C[w1]; kept_M = sh.cut_M[w1]; }
            }
        }
    }
    // the race: every window down to the cut once more, first the one that is counted already
    Cand best = contestant(-1.0f, 0);
    int best_n = 0;
    const int first = resident;
#pragma unroll 1
    for (int i = 0; i < kWideWindows; ++i) {
        const WideWindow win{i == 0 ? first : i <= first ? i - 1 : i};
        if (sh.C_above[win.w + 1] == sh.C_above[win.w] || key_of_pattern(win.pattern(0)) < cut_key) continue;   // uniform
        wide_count(row, win, resident, hist, tid);
        Cand mine = contestant(-1.0f, 0);
#pragma unroll 4
        for (int rank = tid; rank < kWideBins; rank += kRThreads) {
            const uint32_t n = count_of(win, rank);
            const int p = win.pattern(rank);
            if (n != 0u && key_of_pattern(p) >= cut_key)
                mine = better(mine, contestant(level_score(p, (int)n, (float)z1, c, a.seed, grow), key_of_pattern(p)));
        }
        mine = reduce_best(mine, sh, tid);
        const Cand was = best;
        best = better(was, mine);
        if (best.idx != was.idx || best.q != was.q) best_n = (int)hist[wide_place((uint32_t)pattern_of_key(key_of(best)))];
    }
    const bool drawn = best.q >= 0.0f;
    const int pattern = pattern_of_key(key_of(best));
    if (tid == 0) store_row(a, r, kept_C, drawn, pattern, z1, log(kept_M), inv_tau);
    if (drawn) locate<kBlock>(row, 0, 0, row.steps, (uint32_t)pattern, (int)(((2ull * k23 + 1ull) * (uint64_t)best_n) >> 24), a.token_out + r, sh, tid);
}

// ---------------------------------------------------------------------------
// The near window.
// ---------------------------------------------------------------------------
struct Near {
    int base;             // magnitude bits of the window's lowest level
    int per_quarter;      // stream steps per quarter
    float first_top;      // the largest finite value among the first vectors (-inf: none)
    const uint32_t* hist;
    // rank 0 .. kHalf - 1: non-negative levels from the top, then the negative ones.  A word holds two
    // quarters' counters of a level; each sign's words lie in rising magnitude, the highest kTrash of them
    // being the spare ones.
    __device__ __forceinline__ int slot(int rank) const { return rank < kHalf ? kHalf - 1 - rank : rank; }
    __device__ __forceinline__ int slot_of_pattern(int p) const { return (p & 0x7FFF) - base + (p >> 15) * kHalf; }
    __device__ __forceinline__ int pattern(int rank) const
    {
        return rank < kHalf ? base + kHalf - 1 - rank : 0x8000 + base + rank - kHalf;
    }
    static __device__ __forceinline__ int total(uint32_t a, uint32_t b)      // of the four quarters
    {
        return (int)__builtin_amdgcn_sad_u16(b, 0u, __builtin_amdgcn_sad_u16(a, 0u, 0u));
    }
    __device__ __forceinline__ int count(int rank) const { return total(hist[slot(rank)], hist[kArray + slot(rank)]); }
    // the counts of the kOwnN levels from rank0 (a multiple of kOwnN) on
    __device__ __forceinline__ void own_counts(int rank0, int cnt[kOwnN]) const
    {
        const bool neg = __builtin_amdgcn_readfirstlane(rank0) >= kHalf;         // a wave's levels have one sign
        const uint32_t* h = hist + (neg ? rank0 : kHalf - kOwnN - rank0);
        uint32_t sum[kOwnN];                                      // in rising magnitude
        auto from = [&](const uint4& a, const uint4& b, int i) {
            sum[i] = (uint32_t)total(a.x, b.x); sum[i + 1] = (uint32_t)total(a.y, b.y);
            sum[i + 2] = (uint32_t)total(a.z, b.z); sum[i + 3] = (uint32_t)total(a.w, b.w);
        };
        if (kOwnN == 8) {
            // (sixteen waves: each four added as it comes, 256 rows x 151,936 22.7 -> 22.2 us)
#pragma unroll
            for (int i = 0; i < kOwnN; i += 4) from(*reinterpret_cast<const uint4*>(h + i), *reinterpret_cast<const uint4*>(h + kArray + i), i);
        } else {
            uint4 a[kOwnN / 4], b[kOwnN / 4];
#pragma unroll
            for (int i = 0; i < kOwnN / 4; ++i) { a[i] = reinterpret_cast<const uint4*>(h)[i]; b[i] = reinterpret_cast<const uint4*>(h + kArray)[i]; }
#pragma unroll
            for (int i = 0; i < kOwnN / 4; ++i) from(a[i], b[i], 4 * i);
        }
#pragma unroll
        for (int j = 0; j < kOwnN; ++j) cnt[j] = (int)(neg ? sum[j] : sum[kOwnN - 1 - j]);
        static_assert(kTrash % kOwnN == 0, "a thread's words are levels or spare ones");
        if (rank0 < kTrash || rank0 >= 2 * kHalf - kTrash) {
#pragma unroll
            for (int j = 0; j < kOwnN; ++j) cnt[j] = 0;
        }
    }
    // first / last rank whose key is at most / at least `key`
    __device__ __forceinline__ int first_at_most(int key) const
    {
        if (key >= 0x8000 + base + kHalf) return 0;
        if (key >= 0x8000 + base) return 0x8000 + base + kHalf - 1 - key;
        if (key > 0x7FFF - base) return kHalf;
        return kHalf + (0x7FFF - base) - key;
    }
    __device__ __forceinline__ int last_at_least(int key) const
    {
        if (key > 0x8000 + base + kHalf - 1) return -1;
        if (key >= 0x8000 + base) return 0x8000 + base + kHalf - 1 - key;
        if (key > 0x7FFF - base) return kHalf - 1;
        const int r = kHalf + (0x7FFF - base) - key;
        return r < kHalf + kLevels ? r : kHalf + kLevels - 1;
    }
};

// What of a lane's columns lies outside the window, by kind: two 16-bit counts to a word (a lane has at most
// 8 x 2032 columns of the widest row).
struct Tally {
    uint32_t zeros;       // +0, -0, of the current quarter
    uint32_t far;         // columns below the window, above it
    uint32_t odd;         // no numbers
    u16x2 lowest, highest, top;     // (magnitude - window's end) of the columns below the window, wrapped down by one, and as it is; of those above
};

// Patterns of a word at or above c (as unsigned numbers), 0 or 1 in each half.
static __device__ __forceinline__ u16x2 at_least(u16x2 w, uint32_t c)
{
    const uint16_t c1 = (uint16_t)(c - 1u);
    const u16x2 less = {c1, c1}, one = {1, 1};
    return __builtin_elementwise_min(__builtin_elementwise_sub_sat(w, less), one);
}

// A vector step that may hold patterns outside the window (rare): all lanes of the wave take part, a lane with its
// vector, the columns col0, col0 + 1, ..., if `mine`.
static __device__ __forceinline__ void note_outside(const u32x4& x, int col0, bool mine, int quarter, int base, Tally& t, Shared& sh)
{
    const u16x2 base_v = {(uint16_t)base, (uint16_t)base};
    auto level = [&](uint32_t w) -> u16x2 { return halves(__builtin_bit_cast(uint32_t, halves(w) - base_v) & 0x7FFF7FFFu); };
    const u16x2 worst = __builtin_elementwise_max(__builtin_elementwise_max(level(x.x), level(x.y)),
                                                  __builtin_elementwise_max(level(x.z), level(x.w)));
    const bool out = mine && (worst.x >= kLevels || worst.y >= kLevels);
    if (!__any(out)) return;
    auto both = [](u16x2 n) -> int { return (int)n.x + (int)n.y; };
    auto each = [&](auto&& f) { f(x.x); f(x.y); f(x.z); f(x.w); };
    // what is no number (masked columns) is only counted
    u16x2 outside = {0, 0}, odd = {0, 0}, near = {0, 0};          // near: as a count of what is not
    each([&](uint32_t word) {
        outside += at_least(level(word), (uint32_t)kLevels);
        odd += at_least(halves(word & 0x7FFF7FFFu), 0x7F80u);
    });
    const int n_odd = both(odd);
    if (out) t.odd += (uint32_t)n_odd;
    if (!__any(out && both(outside) > n_odd)) return;
    each([&](uint32_t word) { near += at_least(halves(word & 0x7FFF7FFFu), (uint32_t)base); });
    const int n_near = out && base > 0 ? 8 - both(near) : 0;      // base 0: zeros are levels
    if (__any(out && both(outside) > n_odd + n_near)) {
        const uint32_t end = (uint32_t)(base + kLevels);
        const uint16_t end1 = (uint16_t)(end - 1u), neg1 = (uint16_t)(0x8000u + end - 1u);
        const u16x2 e1 = {end1, end1}, n1 = {neg1, neg1}, one = {1, 1};
        u16x2 above = {0, 0}, below = {0, 0};
        if (out) {
            each([&](uint32_t word) {
                const u16x2 w = halves(word);
                const u16x2 is_above = at_least(w, end) - at_least(w, 0x7F80u), is_below = at_least(w, 0x8000u + end) - at_least(w, 0xFF80u);
                above += is_above;
                below += is_below;
                t.top = __builtin_elementwise_max(t.top, __builtin_elementwise_sub_sat(w, e1) * is_above);
                const u16x2 far = __builtin_elementwise_sub_sat(w, n1) * is_below;
                t.highest = __builtin_elementwise_max(t.highest, far);
                t.lowest = __builtin_elementwise_min(t.lowest, far - one);
            });
            t.far += (uint32_t)(both(below) | both(above) << 16);
            if (both(above) != 0) sh.fails = 1;
        }
    }
    if (__any(n_near != 0) && n_near != 0) {
        const u16x2 one = {1, 1};
        u16x2 zero_p = {0, 0}, zero_n = {0, 0};
        each([&](uint32_t word) {
            zero_p += one - at_least(halves(word), 1u);
            zero_n += one - at_least(halves(word ^ 0x80008000u), 1u);
        });
        t.zeros += (uint32_t)(both(zero_p) | both(zero_n) << 16);
        if (n_near != both(zero_p) + both(zero_n)) {              // small values are listed one by one
            u32x4 rest = x;
#pragma unroll 1
            for (int j = 0; j < 8; ++j) {
                const uint32_t p = rest.x & 0xFFFFu, mag = p & 0x7FFFu;
                if (mag != 0u && mag < (uint32_t)base) {
                    const int at = atomicAdd(&sh.list_n, 1);
                    if (at < kMidList) { sh.list_key[at] = key_of_pattern((int)p); sh.list_col[at] = col0 + j; }
                    else sh.fails = 1;
                }
                rest.x = rest.x >> 16 | rest.y << 16; rest.y = rest.y >> 16 | rest.z << 16;
                rest.z = rest.z >> 16 | rest.w << 16; rest.w >>= 16;
            }
        }
    }
}

// The zeros of a quarter, and at the end the rest, to the workgroup.
static __device__ __forceinline__ void hand_zeros(Tally& t, int quarter, Shared& sh, int lane)
{
    if (!__any(t.zeros != 0u)) return;
    const uint32_t p = (uint32_t)wave_prefix_sum((int)(t.zeros & 0xFFFFu)), n = (uint32_t)wave_prefix_sum((int)(t.zeros >> 16));
    if (lane == 63) { atomicAdd(&sh.zeros[0][quarter], (int)p); atomicAdd(&sh.zeros[1][quarter], (int)n); }
    t.zeros = 0u;
}
static __device__ __forceinline__ void hand_rest(const Tally& t, int base, Shared& sh, int lane)
{
    if (!__any((t.far | t.odd) != 0u)) return;
    const int below = wave_prefix_sum((int)(t.far & 0xFFFFu)), above = wave_prefix_sum((int)(t.far >> 16)), odd = wave_prefix_sum((int)t.odd);
    if (lane == 63) { atomicAdd(&sh.n_below, below); atomicAdd(&sh.n_above, above); atomicAdd(&sh.n_not_finite, odd); }
    const int end1 = base + kLevels - 1;
    auto most = [](u16x2 a) -> float { return (float)(a.x > a.y ? a.x : a.y); };
    const float top = wave_max(most(t.top)), hi = wave_max(most(t.highest));
    const float lo = -wave_max(-(float)(t.lowest.x < t.lowest.y ? t.lowest.x : t.lowest.y));
    if (lane == 0) {
        if (top > 0.0f) atomicMax(&sh.above_hi, end1 + (int)top);
        if (hi > 0.0f) { atomicMax(&sh.below_hi, end1 + (int)hi); atomicMin(&sh.below_lo, end1 + 1 + (int)lo); }
    }
}

// The largest finite value among a wave's first vectors, -inf if there is none.  As signed 16-bit integers
// the patterns of non-negative values are in value order above all others; a wave without any, or with an
// infinity or a NaN on top, looks through its values one by one.
template <int kN, typename Get>
static __device__ __forceinline__ float wave_top_value(Get&& get)
{
    s16x2 m = {-32768, -32768};
#pragma unroll
    for (int u = 0; u < kN; ++u) {
        const u32x4 v = get(u);
        m = __builtin_elementwise_max(m, __builtin_elementwise_max(signed_halves(v.x), signed_halves(v.y)));
        m = __builtin_elementwise_max(m, __builtin_elementwise_max(signed_halves(v.z), signed_halves(v.w)));
    }
    const float best = wave_max((float)(m.x > m.y ? m.x : m.y));
    if (__builtin_expect(best >= 0.0f && best < (float)0x7F80, 1)) return value_of_pattern((int)best);     // uniform
    float f = -INFINITY;
#pragma unroll
    for (int u = 0; u < kN; ++u)
        for_each_pattern(get(u), [&](uint32_t p, int) {
            const float z = value_of_pattern((int)p);
            f = z < INFINITY ? fmaxf(f, z) : f;
        });
    return wave_max(f);
}

// The top binade of a window lowered for a row of which `mag` is the largest magnitude seen.
static __device__ __forceinline__ int lowered_top(float mag) { return (int)(__float_as_uint(mag) >> 23) + 12; }

// Counts the row.  Returns the window, whose top binade is `top_exp` if that is not negative.  Two sets of
// requests are in flight: a set is asked for as soon as the one before it in its registers is counted.
// kSlice: `row` is a slice, from column col0 on, of `whole`, and counts as one quarter; the window then follows from 64
// vectors spread over the whole row, the same ones for all its slices, and is lowered where they are small.
template <bool kSlice>
static __device__ __forceinline__ Near near_count(const Row& row, const Row& whole, int col0, int top_exp, uint32_t* hist,
                                                  Shared& sh, int tid)
{
    const int lane = tid & 63, wave = tid >> 6;
    Near w;
    w.hist = hist;
    w.per_quarter = kSlice ? 1 << 30 : (row.steps + kQuarters - 1) / kQuarters;
    u32x4 x[kSet], y[kSet], spread{0u, 0u, 0u, 0u};
    const int spread_at = kSlice ? (int)((int64_t)whole.nvec * lane / 64) : 0;
    if (kSlice && wave == 0) spread = whole.p[spread_at];
    row.template request_ahead<kSet>(x, 0, tid);
    row.template request_ahead<kSet>(y, kSet, tid);
    uint32_t tail = 0u;                                           // the columns behind the last complete vector
    if (row.last < 8 && tid < row.last) tail = reinterpret_cast<const uint16_t*>(row.p + row.complete)[tid];
    for (int i = tid; i < (kSlice ? 1 : 2) * kArray / 4; i += kRThreads) reinterpret_cast<uint4*>(hist)[i] = uint4{0u, 0u, 0u, 0u};
    if (tid < 2 * kQuarters) (&sh.zeros[0][0])[tid] = 0;
    if (tid == 0) {
        sh.list_n = 0; sh.n_below = 0; sh.n_not_finite = 0; sh.n_above = 0;
        sh.below_lo = 0x7FFF; sh.below_hi = 0; sh.above_hi = 0; sh.fails = 0;
    }
    {
        const float m = kSlice
            ? wave == 0 ? wave_top_value<1>([&](int) { return whole.counted(spread, spread_at); }) : -INFINITY
            : wave_top_value<2 * kSet>([&](int u) {
                  const u32x4 v = u < kSet ? x[u % kSet] : y[u % kSet];
                  return u < row.whole ? v : row.counted(v, tid + u * kRThreads);
              });
        if (lane == 0) sh.sample_max[wave] = m;
        if (kSlice && wave == 0 && m >= 0.0f && lowered_top(m) < kTopExp) {                // uniform, rare
            const u32x4 v = whole.counted(spread, spread_at);
            const u16x2 one = {1, 1};
            auto held = [&](uint32_t word) -> u16x2 {
                const u16x2 mag = halves(word & 0x7FFF7FFFu);
                return mag * (one - at_least(mag, (uint32_t)kTopEnd));
            };
            const u16x2 most = __builtin_elementwise_max(__builtin_elementwise_max(held(v.x), held(v.y)),
                                                         __builtin_elementwise_max(held(v.z), held(v.w)));
            const float mag = wave_max((float)(most.x > most.y ? most.x : most.y));
            if (lane == 0) sh.sample_mag = value_of_pattern((int)mag);
        }
    }
    // orders LDS only: __syncthreads() would wait for the loads in flight as well
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    w.first_top = row16_max(sh.sample_max[lane & (kRWaves - 1)]);
    // the window's top: one binade above the magnitude of the largest finite logit among the first
    // vectors (if that is negative, up to 2^20: what lies far down is a mask)
    if (top_exp < 0) {
        top_exp = w.first_top > -1048576.0f ? (int)(__float_as_uint(fabsf(w.first_top)) >> 23) + 1 : 0;
        // (lowered only for a non-negative value, and to eleven binades above all that the sample holds of either
        // sign: half of a row at zero and the others negative is an ordinary row)
        int least = kTopExp;
        if (kSlice && w.first_top >= 0.0f && lowered_top(w.first_top) < kTopExp) {
            const int lower = lowered_top(sh.sample_mag);
            least = lower < kTopExp ? lower : kTopExp;
        }
        top_exp = top_exp < least ? least : top_exp;
    }
    top_exp = top_exp > 254 ? 254 : top_exp < kBinades - 1 ? kBinades - 1 : top_exp;
    w.base = __builtin_amdgcn_readfirstlane(top_exp > kBinades - 1 ? ((top_exp - (kBinades - 1)) << 7) + kTrash : 0);

    // Two patterns at a time: less the window's base, and without the sign, the magnitude is the level, and
    // anything outside the window (wrapped around or past the end) is a large number that a minimum
    // sends to the lane's own spare word; the sign goes next to the twelve bits of the level.  Five packed
    // or plain instructions per column with the two addresses.
    static_assert(kHalf == 4096 && kArray * 4 == 0x8000, "places of 13 bits, the array next to them");
    const uint16_t base1 = (uint16_t)w.base, spare = (uint16_t)(kLevels + lane);
    const u16x2 base_v = {base1, base1}, spare_v = {spare, spare};
    u16x2 worst = {0, 0};
    auto add8 = [&](const u32x4& x, int step) {
        const int quarter = step / w.per_quarter;
        const uint32_t array = (uint32_t)(quarter >> 1) << 15, inc = 1u << ((quarter & 1) * 16);
        char* h = reinterpret_cast<char*>(hist);
        auto add2 = [&](uint32_t word) {
            const uint32_t s = __builtin_bit_cast(uint32_t, halves(word) - base_v);
            const u16x2 level = halves(s & 0x7FFF7FFFu);
            worst = __builtin_elementwise_max(worst, level);
            const uint32_t at = __builtin_bit_cast(uint32_t, __builtin_elementwise_min(level, spare_v)) | (s >> 3 & 0x10001000u);
            atomicAdd(reinterpret_cast<uint32_t*>(h + ((at << 2 & 0x7FFCu) | array)), inc);
            atomicAdd(reinterpret_cast<uint32_t*>(h + ((at >> 14 & 0x7FFCu) | array)), inc);
        };
        add2(x.x); add2(x.y); add2(x.z); add2(x.w);
    };
    Tally t{0u, 0u, 0u, {0xFFFF, 0xFFFF}, {0, 0}, {0, 0}};
    int noted = 0;                                                // the quarter of t.zeros
    auto note = [&](const u32x4& y, int step, int col0, bool mine) {
        const int quarter = step / w.per_quarter;
        if (quarter != noted) { hand_zeros(t, noted, sh, lane); noted = quarter; }
        note_outside(y, col0, mine, quarter, w.base, t, sh);
    };
    auto count = [&](const u32x4 (&x)[kSet], int i0) -> bool {
        worst = u16x2{0, 0};
#pragma unroll
        for (int u = 0; u < kSet; ++u) {
            if (tid + (i0 + u) * kRThreads < row.complete) add8(x[u], i0 + u);
        }
        if (__builtin_expect(!__any(worst.x >= kLevels || worst.y >= kLevels), 1)) return false;
#pragma unroll 1
        for (int u = 0; u < kSet; ++u) {
            u32x4 y = x[0];
#pragma unroll
            for (int i = 1; i < kSet; ++i) {
                const uint32_t is = i == u ? 0xFFFFFFFFu : 0u;
                y = (y & ~is) | (x[i] & is);
            }
            const int v = tid + (i0 + u) * kRThreads;
            note(y, i0 + u, col0 + v * 8, v < row.complete);
        }
        return __builtin_amdgcn_readfirstlane(*(volatile int*)&sh.fails) != 0;             // counted enough
    };
    for (int i0 = 0;; i0 += 2 * kSet) {
        if (count(x, i0) || i0 + kSet >= row.steps) break;
        row.template request_ahead<kSet>(x, i0 + 2 * kSet, tid);
        if (count(y, i0 + kSet) || i0 + 2 * kSet >= row.steps) break;
        row.template request_ahead<kSet>(y, i0 + 3 * kSet, tid);
    }
    if (row.last < 8 && wave == 0) {                              // the row's last columns, one per lane
        const bool mine = lane < row.last;
        const uint32_t level = (tail & 0x7FFFu) - (uint32_t)w.base, inside = (uint32_t)w.base * 0x10001u;
        const int quarter = (row.steps - 1) / w.per_quarter;
        if (mine && level < (uint32_t)kLevels)
            atomicAdd(&hist[(quarter >> 1) * kArray + level + (tail >> 15) * kHalf], 1u << ((quarter & 1) * 16));
        if (__any(mine && level >= (uint32_t)kLevels))
            note(u32x4{tail | (inside & 0xFFFF0000u), inside, inside, inside}, row.steps - 1, col0 + row.complete * 8 + lane, mine);
    }
    hand_zeros(t, noted, sh, lane);
    hand_rest(t, w.base, sh, lane);
    __syncthreads();
    return w;
}

// Counts the row, into a second window if the first had columns above it or too many small ones:
// four binades above the largest it has seen (its waves stop at the first), or three above the
// largest among the first vectors.  top_exp: the window's top binade where it is known already, or -1.
static __device__ __forceinline__ Near near_window(const Row& row, int top_exp, uint32_t* hist, Shared& sh, int tid)
{
    Near w;
#pragma unroll 1
    for (;;) {
        int me = tid;
        Row again = row;
        // Opaque copies: otherwise the compiler holds what it can share between the two counts in
        // registers, and the stream spills (512 rows 45 -> 51 us).
        asm volatile("" : "+v"(me), "+s"(again.nvec), "+s"(again.last), "+s"(again.steps), "+s"(again.whole), "+s"(again.complete));
        w = near_count<false>(again, again, 0, top_exp, hist, sh, me);
        if (__builtin_expect(sh.fails == 0 || top_exp >= 0, 1)) return w;                 // uniform
        const int now = (w.base >> 7) + kBinades - 1;
        if (sh.n_above != 0) {
            top_exp = (sh.above_hi >> 7) + 4;
        } else {
            top_exp = (int)((__float_as_uint(w.first_top) >> 23) & 0xFFu) + 3;
            if (top_exp > now - 8) return w;                      // hardly lower: the small values lie below it as well
        }
        top_exp = __builtin_amdgcn_readfirstlane(top_exp);
        __syncthreads();
    }
}

// One slice of a row: its counters, 16 bits each, and its notes go to memory.
static __device__ __forceinline__ void count_slice(const RestrictedArgs& a, uint32_t* hist, Shared& sh)
{
    const int tid = threadIdx.x;
    const int64_t r = blockIdx.x / a.nslices;
    const int s = blockIdx.x - (int)r * a.nslices;
    const Row row = whole_row(a, r);
    const int v0 = row.slice_begin(s, a.nslices);
    const Near w = near_count<true>(row.part(v0, row.slice_begin(s + 1, a.nslices)), row, v0 * 8, -1, hist, sh, tid);
    uint32_t packed[kOwnN / 2];
#pragma unroll
    for (int i = 0; i < kOwnN; i += 4) {
        const uint4 c = *reinterpret_cast<const uint4*>(hist + kOwnN * tid + i);
        packed[i / 2] = c.x | c.y << 16;
        packed[i / 2 + 1] = c.z | c.w << 16;
    }
    uint32_t* out = reinterpret_cast<uint32_t*>(a.slice_counts + (size_t)blockIdx.x * kArray + kOwnN * tid);
#pragma unroll
    for (int i = 0; i < kOwnN / 2; i += 4)
        *reinterpret_cast<uint4*>(out + i) = uint4{packed[i], packed[i + 1], packed[i + 2], packed[i + 3]};
    SliceNotes& n = a.slice_notes[blockIdx.x];
    const int listed = sh.list_n < kMidList ? sh.list_n : kMidList;
    if (tid == 0) {
        n.zeros[0] = sh.zeros[0][0]; n.zeros[1] = sh.zeros[1][0];
        n.list_n = sh.list_n; n.n_below = sh.n_below; n.n_not_finite = sh.n_not_finite;
        n.below_lo = sh.below_lo; n.below_hi = sh.below_hi; n.above_hi = sh.above_hi;
        n.base = w.base; n.first_top = w.first_top;
    }
    if (tid < listed) { n.list_key[tid] = sh.list_key[tid]; n.list_col[tid] = sh.list_col[tid]; }
}

// The counters and notes of a row's slices, as near_window leaves those of a row it has counted itself, and -1; or the top
// binade of the window that the row is to be counted in instead, by the rules of near_window.
static __device__ __forceinline__ int gather_slices(const RestrictedArgs& a, int64_t r, Near& w, uint32_t* hist, Shared& sh, int tid)
{
    const int lane = tid & 63, wave = tid >> 6, per = a.nslices / kQuarters;
    const uint16_t* counts = a.slice_counts + (size_t)r * a.nslices * kArray + kOwnN * tid;
    w.hist = hist;
    w.per_quarter = 0;
    // a quarter is `per` slices; a thread sums the two quarters of one array at a time, two levels per word (a sum past
    // 16 bits reaches the next level, and the counts no longer add up to the row's width)
#pragma unroll 1
    for (int array = 0; array < 2; ++array) {
        uint32_t sum[2][kOwnN / 2] = {};
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            if (s >= per) break;                                  // uniform
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const uint4* from = reinterpret_cast<const uint4*>(counts + (size_t)((2 * array + q) * per + s) * kArray);
#pragma unroll
                for (int i = 0; i < kOwnN / 8; ++i) {
                    const uint4 c = from[i];
                    sum[q][4 * i] += c.x; sum[q][4 * i + 1] += c.y; sum[q][4 * i + 2] += c.z; sum[q][4 * i + 3] += c.w;
                }
            }
        }
        uint32_t* to = hist + array * kArray + kOwnN * tid;
#pragma unroll
        for (int i = 0; i < kOwnN / 2; i += 2) {
            uint4 c;
            c.x = (sum[0][i] & 0xFFFFu) | sum[1][i] << 16; c.y = sum[0][i] >> 16 | (sum[1][i] & 0xFFFF0000u);
            c.z = (sum[0][i + 1] & 0xFFFFu) | sum[1][i + 1] << 16; c.w = sum[0][i + 1] >> 16 | (sum[1][i + 1] & 0xFFFF0000u);
            *reinterpret_cast<uint4*>(to + 2 * i) = c;
        }
    }
    if (wave == 0) {
        const SliceNotes* n = a.slice_notes + r * a.nslices + (lane < a.nslices ? lane : 0);
        const bool mine = lane < a.nslices;
        const int list_n = mine ? n->list_n : 0;
        const int outside = mine ? list_n | n->zeros[0] | n->zeros[1] | n->n_below | n->n_not_finite | n->above_hi : 0;
        if (!__any(outside != 0)) {                               // an ordinary row (8 x 151,936 14.8 -> 14.2 us without the sums)
            if (lane < 2 * kQuarters) (&sh.zeros[0][0])[lane] = 0;
            if (lane == 0) {
                sh.list_n = 0; sh.n_below = 0; sh.n_not_finite = 0; sh.n_above = 0;
                sh.below_lo = 0x7FFF; sh.below_hi = 0; sh.above_hi = 0;
            }
        } else {
            const int lists = wave_prefix_sum(list_n);
            const int zero_p = wave_prefix_sum(mine ? n->zeros[0] : 0), zero_n = wave_prefix_sum(mine ? n->zeros[1] : 0);
            const int below = wave_prefix_sum(mine ? n->n_below : 0), odd = wave_prefix_sum(mine ? n->n_not_finite : 0);
            const float lo = -wave_max(mine ? -(float)n->below_lo : -32767.0f), hi = wave_max(mine ? (float)n->below_hi : 0.0f);
            const int above = (int)wave_max(mine ? (float)n->above_hi : 0.0f), all_listed = __builtin_amdgcn_readlane(lists, 63);
            if (lane == 63) {
                sh.zeros[0][0] = zero_p; sh.zeros[1][0] = zero_n;
                sh.list_n = lists; sh.n_below = below; sh.n_not_finite = odd; sh.n_above = 0;
                sh.below_lo = (int)lo; sh.below_hi = (int)hi; sh.above_hi = above;
            }
            if (lane > 0 && lane < kQuarters) { sh.zeros[0][lane] = 0; sh.zeros[1][lane] = 0; }
            if (all_listed <= kMidList) {
                for (int i = 0; i < list_n; ++i) {
                    sh.list_key[lists - list_n + i] = n->list_key[i];
                    sh.list_col[lists - list_n + i] = n->list_col[i];
                }
            }
        }
    }
    const SliceNotes& first = a.slice_notes[r * a.nslices];
    w.base = __builtin_amdgcn_readfirstlane(first.base);
    w.first_top = uniform_f(first.first_top);
    __syncthreads();
    int top_exp = -1;
    if (sh.above_hi != 0) {
        top_exp = (sh.above_hi >> 7) + 4;
    } else if (sh.list_n > kMidList) {                            // (not lower: such a row takes the wide form)
        const int lower = (int)((__float_as_uint(w.first_top) >> 23) & 0xFFu) + 3;
        if (lower <= (w.base >> 7) + kBinades - 1 - 8) top_exp = lower;
    }
    // columns below a lowered window that the ordinary one holds (the sample had none of them): the lowest window that does
    if (sh.n_below != 0 && sh.below_lo < kTopEnd) {
        const int reach = sh.below_hi < kTopEnd ? sh.below_hi >> 7 : kTopExp;
        top_exp = top_exp < reach ? reach : top_exp;
    }
    __syncthreads();                                              // what was read here may be counted anew
    return __builtin_amdgcn_readfirstlane(top_exp);
}

// The middle items of a row, one per lane of one wave, in rank order: the listed small
// positive values, +0, -0, the small negative ones.
static __device__ __forceinline__ void middle_items(Shared& sh, int lane)
{
    const int n = sh.list_n;
    const int key = lane < n ? sh.list_key[lane] : 0, col = lane < n ? sh.list_col[lane] : 0;
    int rank = 0;
    for (int e = 0; e < n; ++e) {
        const int ok = __builtin_amdgcn_readlane(key, e), oc = __builtin_amdgcn_readlane(col, e);
        rank += ok > key || (ok == key && oc < col);
    }
    const int npos = __popcll(__ballot(lane < n && key > 0x8000));
    if (lane < n) {
        const int at = rank < npos ? rank : rank + 2;
        sh.mid_key[at] = key; sh.mid_cnt[at] = 1; sh.mid_col[at] = col;
    }
    if (lane < 2) {
        int c = 0;
        for (int q = 0; q < kQuarters; ++q) c += sh.zeros[lane][q];
        sh.mid_key[npos + lane] = 0x8000 - lane; sh.mid_cnt[npos + lane] = c; sh.mid_col[npos + lane] = -1;
    }
}

// kCut: the row's slices have been counted.
template <bool kCut>
static __device__ __forceinline__ void run(const RestrictedArgs& a, uint32_t* hist, Shared& sh)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t r = blockIdx.x;
    const Row row = whole_row(a, r);
    const float tau = a.tau_rows ? a.tau_rows[r] : a.tau_scalar;
    const double inv_tau = 1.0 / (double)tau;
    const float c = kLog2eF / tau;
    const uint64_t grow = a.row_base + (uint64_t)r;
    const bool k_on = a.top_k >= 1 && (int64_t)a.top_k < a.V, p_on = a.top_p < 1.0f;

    uint32_t k23;                                                 // picks the column within the winning level
    {
        uint32_t w4[4];
        philox4x32_10(0u, (uint32_t)grow, (uint32_t)(grow >> 32), 4u, (uint32_t)a.seed, (uint32_t)(a.seed >> 32), w4);
        k23 = w4[0] >> 9;
    }
    Near win;
    const int anew = kCut ? gather_slices(a, r, win, hist, sh, tid) : -1;
    const bool sliced = kCut && anew < 0;                         // uniform
    if (!sliced) win = near_window(row, anew, hist, sh, tid);

    const int list_n = sh.list_n;
    int n_zero = 0;
#pragma unroll
    for (int q = 0; q < 2 * kQuarters; ++q) n_zero += (&sh.zeros[0][0])[q];
    const bool listed = list_n <= kMidList;
    const bool has_mid = listed && (n_zero != 0 || list_n != 0);
    const int n_mid = has_mid ? list_n + 2 : 0;
    if (has_mid && wave == 0) {
        middle_items(sh, lane);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
    // Masses and the scan; the middle comes between the two signs.  The weights are relative to the first
    // vectors' largest value, so that the row's largest needs no barrier of its own; if that is so much
    // larger that they could overflow, once more relative to it.
    View vw;
    const int rank0 = kOwnN * tid;
    double z_ref = (double)win.first_top, z1, M_win;
    float top_key;
    int C_win;
    bool again = false;
#pragma unroll 1
    for (;;) {
        // my levels, and the row's highest one
        int cnt[kOwnN];
        win.own_counts(rank0, cnt);
        vw.Cl = 0; vw.top = kOwnN;
#pragma unroll
        for (int j = kOwnN - 1; j >= 0; --j) {
            vw.Cl += cnt[j];
            if (cnt[j] != 0) vw.top = j;
        }
        const int p_top = win.pattern(rank0 + (vw.Cl > 0 ? vw.top : 0));
        int top = vw.Cl > 0 ? key_of_pattern(p_top) : -1;
        if (has_mid && wave == 0 && lane < n_mid && sh.mid_cnt[lane] != 0 && sh.mid_key[lane] > top) top = sh.mid_key[lane];
        const float wave_top = wave_max((float)top);              // keys are below 2^16: exact in fp32
        if (lane == 0) sh.wave_top[wave] = wave_top;
        own_mass<kOwnN, kOwnN>(vw, (p_top >> 7) & 0xFF, value_of_pattern(p_top), z_ref, inv_tau, [&](int j) { return cnt[j]; });
        if (has_mid && wave == 0) {
            const int n = lane < n_mid ? sh.mid_cnt[lane] : 0;
            const double w = n != 0 ? exp(((double)value_of_pattern(pattern_of_key(sh.mid_key[lane])) - z_ref) * inv_tau) : 0.0;
            sh.mid_C[lane] = wave_prefix_sum(n);
            sh.mid_M[lane] = wave_prefix_sum((double)n * w);
        }
        const Waves all = scan_view(vw, 0, 0.0, has_mid ? kRThreads / 2 : kRThreads, sh, tid);
        C_win = __builtin_amdgcn_readlane(all.C, kRWaves - 1); M_win = read_lane(all.M, kRWaves - 1);
        top_key = row16_max(sh.wave_top[lane & (kRWaves - 1)]);
        z1 = top_key >= 0.0f ? (double)value_of_pattern(pattern_of_key((int)top_key)) : 0.0;
        if (again || fabs((z1 - z_ref) * inv_tau) < 256.0) break;                // uniform
        __syncthreads();
        again = true;
        z_ref = z1;
    }
    const float z1f = (float)z1;                                  // a bf16 value: exact
    const int mid_C = has_mid ? sh.mid_C[63] : 0;
    const double mid_M = has_mid ? sh.mid_M[63] : 0.0;
    const int n_below = sh.n_below;
    const int C_in = C_win + mid_C, C_all = C_in + n_below;
    const double M_all = M_win + mid_M;

    // Columns below the window weigh nothing when every one of them is below 2^-80 of the largest
    // weight: a row of them stays below the last bit of the total, which is at least 1, and none can win the race.
    const bool below_weightless = n_below == 0
        || (top_key >= 0.0f && (-(double)value_of_pattern(sh.below_lo) - z1) * inv_tau < -56.0);
    const bool wide = sh.n_above != 0 || !listed || !below_weightless
             || C_win + n_zero + list_n + n_below + sh.n_not_finite + sh.n_above != (int)a.V                       // a counter wrapped
             || (k_on && C_all >= a.top_k && C_in < a.top_k && sh.below_lo != sh.below_hi);           // the cut is below the window
    if (wide) {                                                   // uniform
        wide_row(row, a, r, inv_tau, c, grow, k23, hist, sh, tid);
    } else if (top_key >= 0.0f) {
        int cut_key = 0, kept_C = C_all;
        double kept_M = M_all;
        auto my_cnt = [&](int j) { return win.count(rank0 + j); };
        auto my_key = [&](int j) { return key_of_pattern(win.pattern(rank0 + j)); };
        // The middle's share of a search, by the first negative wave: the items carry inclusive
        // prefixes; what lies above them is what the wave's first thread has above it, less the middle.
        constexpr int kMidWave = kRWaves / 2;
        int C0 = 0;
        double M0 = 0.0;
        bool level_end = false;
        if (has_mid && wave == kMidWave) {
            C0 = __builtin_amdgcn_readfirstlane(vw.Cx) - mid_C;
            M0 = read_lane(vw.Mx, 0) - mid_M;
            level_end = lane < n_mid && sh.mid_cnt[lane] != 0
                     && (lane == n_mid - 1 || sh.mid_key[lane + 1] != sh.mid_key[lane]);
        }
        auto offer_middle = [&](bool reaches) {
            const unsigned long long hit = __ballot(level_end && reaches);
            if (hit == 0ull) { if (lane == 0) sh.cut_key[kRWaves] = -1; }
            else if (lane == (int)__builtin_ctzll(hit)) {
                sh.cut_key[kRWaves] = sh.mid_key[lane]; sh.cut_C[kRWaves] = C0 + sh.mid_C[lane]; sh.cut_M[kRWaves] = M0 + sh.mid_M[lane];
            }
        };
        auto take = [&](int w) {
            if (sh.cut_key[w] > cut_key) { cut_key = sh.cut_key[w]; kept_C = sh.cut_C[w]; kept_M = sh.cut_M[w]; }
        };
        if (k_on && C_in >= a.top_k) {                            // exactly one place holds the cut
            if (vw.Cx < a.top_k && vw.Cx + vw.Cl >= a.top_k) {
                const Cut cut = own_count_cut<kOwnN, 1>(vw, a.top_k, my_cnt);
                sh.cut_key[0] = my_key(cut.j); sh.cut_C[0] = cut.C; sh.cut_M[0] = cut.M;
            }
            bool in_mid = false;
            if (has_mid) {
                if (wave == kMidWave) offer_middle(C0 + sh.mid_C[lane] >= a.top_k && C0 < a.top_k);
                __syncthreads();
                in_mid = sh.cut_key[kRWaves] >= 0;
            } else {
                __syncthreads();
            }
            take(in_mid ? kRWaves : 0);
            __syncthreads();
        }
        if (p_on) {
            const double T = (double)a.top_p * kept_M;
            offer_mass_cut<kOwnN>(vw, T, [&](int rank) { return win.count(rank); },
                                  [&](int rank) { return key_of_pattern(win.pattern(rank)); }, sh, tid);
            if (has_mid && wave == kMidWave) offer_middle(M0 + sh.mid_M[lane] >= T);
            __syncthreads();
            const int w1 = first_offer(sh, lane);                 // kRWaves: nobody reaches T, nothing is cut
            if (has_mid && w1 >= kMidWave && sh.cut_key[kRWaves] >= 0) take(kRWaves);
            else if (w1 < kRWaves) take(w1);
        }
        // the race: the kept levels dealt round-robin, so that a short run of them spreads over threads
        Cand best = contestant(-1.0f, 0);
        const double ln_M = wave == kRWaves - 1 ? log(kept_M) : 0.0;         // the wave with the least of the race
        const int last = win.last_at_least(cut_key);
        for (int rank = win.first_at_most((int)top_key) + tid; rank <= last; rank += kRThreads) {
            const int n = win.count(rank);
            if (n != 0) {
                const int p = win.pattern(rank);
                best = better(best, contestant(level_score(p, n, z1f, c, a.seed, grow), key_of_pattern(p)));
            }
        }
        if (has_mid && wave == kRWaves - 1 && lane < n_mid && sh.mid_cnt[lane] != 0) {
            const int key = sh.mid_key[lane];
            if (key >= cut_key && (lane == 0 || sh.mid_key[lane - 1] != key)) {
                int n = sh.mid_cnt[lane];
                for (int e = lane + 1; e < n_mid && sh.mid_key[e] == key; ++e) n += sh.mid_cnt[e];
                best = better(best, contestant(level_score(pattern_of_key(key), n, z1f, c, a.seed, grow), key));
            }
        }
        best = reduce_best(best, sh, tid);

        // the column inside the winning level
        const bool drawn = best.q >= 0.0f;
        const int pattern = pattern_of_key(key_of(best)), mag = pattern & 0x7FFF;
        if (tid == kRThreads - 64) store_row(a, r, kept_C, drawn, pattern, z_ref, ln_M, inv_tau);
        auto pick = [&](int n) -> int { return (int)(((2ull * k23 + 1ull) * (uint64_t)n) >> 24); };
        if (drawn && mag != 0 && mag < win.base) {                // a listed value
            if (tid == 0) {
                int at = 0, n = 0;
                for (int e = n_mid - 1; e >= 0; --e)
                    if (sh.mid_key[e] == key_of(best)) { at = e; ++n; }
                a.token_out[r] = sh.mid_col[at + pick(n)];
            }
        } else if (kCut && sliced && drawn) {
            // the slice that holds the column: a lane has a slice's count of the level
            int n = 0;
            if (lane < a.nslices)
                n = mag < win.base ? a.slice_notes[r * a.nslices + lane].zeros[pattern >> 15]
                                   : a.slice_counts[((size_t)r * a.nslices + lane) * kArray + win.slot_of_pattern(pattern)];
            const int upto = wave_prefix_sum(n);
            const int rem = pick(__builtin_amdgcn_readlane(upto, 63));
            const unsigned long long past = __ballot(upto > rem);
            const int s = past != 0ull ? (int)__builtin_ctzll(past) : 0;
            const int v0 = row.slice_begin(s, a.nslices);
            const Row part = row.part(v0, row.slice_begin(s + 1, a.nslices));
            locate<2048 / kRThreads>(part, v0 * 8, 0, part.steps, (uint32_t)pattern, rem - __builtin_amdgcn_readlane(upto - n, s), a.token_out + r, sh, tid);
        } else if (drawn) {
            int q4[kQuarters];
            if (mag < win.base) {                                 // a zero
#pragma unroll
                for (int q = 0; q < kQuarters; ++q) q4[q] = sh.zeros[pattern >> 15][q];
            } else {
                const int s = win.slot_of_pattern(pattern);
                const uint32_t lo = hist[s], hi = hist[kArray + s];
                q4[0] = (int)(lo & 0xFFFFu); q4[1] = (int)(lo >> 16);
                q4[2] = (int)(hi & 0xFFFFu); q4[3] = (int)(hi >> 16);
            }
            int rem = pick(q4[0] + q4[1] + q4[2] + q4[3]), quarter = 0;
#pragma unroll
            for (int q = 0; q < kQuarters - 1; ++q)
                if (quarter == q && rem >= q4[q]) { rem -= q4[q]; ++quarter; }
            const int i0 = quarter * win.per_quarter;
            const int i1 = i0 + win.per_quarter < row.steps ? i0 + win.per_quarter : row.steps;
            // A block that lies past the quarter for the most part costs its requests and comparisons all the same: 512 x
            // 32,000 17.6 us with the one block, 16.4 so.  (A third of half the block: 200 x 60,000 14.8 -> 14.3, but its code
            // cost other widths 0.1 to 0.2 us.)
            if (kRThreads == 512 && i1 - i0 <= kShortBlock)
                locate<kShortBlock>(row, 0, i0, i1, (uint32_t)pattern, rem, a.token_out + r, sh, tid);
            else
                locate<kBlock>(row, 0, i0, i1, (uint32_t)pattern, rem, a.token_out + r, sh, tid);
        }
    } else if (tid == 0) {                                        // no finite logit
        store_row(a, r, 0, false, 0, 0.0, 0.0, inv_tau);
    }
}
};

// Two workgroups of 512 threads per compute unit, or one of 1024: four waves per SIMD, 128 vector registers each.
template <int kRThreads, bool kCut>
__global__ __launch_bounds__(kRThreads, 4)
void sample_restricted_kernel(RestrictedArgs a)
{
    __shared__ __align__(16) uint32_t hist[2 * kArray + kTrash];
    __shared__ typename Sampler<kRThreads>::Shared sh;
    Sampler<kRThreads>::template run<kCut>(a, hist, sh);
}

constexpr int kSliceThreads = 512;
__global__ __launch_bounds__(kSliceThreads, 4)
void count_slices_kernel(RestrictedArgs a)
{
    __shared__ __align__(16) uint32_t hist[kArray];
    __shared__ Sampler<kSliceThreads>::Shared sh;
    Sampler<kSliceThreads>::count_slice(a, hist, sh);
}

}  // namespace

// From this width on a row alone on its compute unit is streamed by sixteen waves (figures: top of this file).
constexpr int64_t kFewWide = 114'688;

// Slices of a row, 0: not cut.  Eight (sixteen where the columns of an eighth would not fit 16-bit counters) for rows of at
// least kSliceMinV columns and 4096 columns per row of the batch, as long as eighths would make at most two workgroups per
// compute unit: what a cut row saves is its stream, what it costs is a launch and 16 KiB of counters per slice.  Whole / eight
// slices / sixteen / four in us: 8 x 151,936 19.4 / 14.9 / 15.9 / 16.6, 32 x 151,936 19.9 / 17.6 / 20.7 / 18.2, 64 x 151,936
// 20.3 / 20.5; 16 x 70,000 15.0 / 14.3, 32 x 70,000 14.9 / 15.6.  (The line follows these widths; wider rows would bear more
// of them: 64 x 260,000, which it leaves whole, 28.1 / 22.6.)
constexpr int64_t kSliceMinV = 65'536;
static int slices_of(int64_t rows, int64_t V)
{
    if (rows < 1 || V < kSliceMinV || rows * 4096 > V || rows * 8 > 2 * (int64_t)compute_units()) return 0;
    return V <= 8 * 65'528 ? 8 : 16;
}

size_t sample_restricted_workspace_bytes(int64_t rows, int64_t V)
{
    return (size_t)rows * slices_of(rows, V) * (kArray * sizeof(uint16_t) + sizeof(SliceNotes));
}

hipError_t launch_sample_restricted(const void* logits, int64_t rows, int64_t V, int64_t row_stride,
                                    const float* tau_rows, float tau_scalar, int32_t top_k, float top_p,
                                    uint64_t seed, uint64_t row_base, int32_t* token_out,
                                    float* logp_out, int32_t* kept_out, void* workspace, size_t workspace_bytes,
                                    hipStream_t stream)
{
    if (rows == 0) return hipSuccess;
    RestrictedArgs a;
    a.logits = static_cast<const uint16_t*>(logits);
    a.rows = rows; a.V = V; a.row_stride = row_stride;
    a.tau_rows = tau_rows; a.tau_scalar = tau_scalar;
    a.top_k = top_k; a.top_p = top_p;
    a.seed = seed; a.row_base = row_base;
    a.token_out = token_out; a.logp_out = logp_out; a.kept_out = kept_out;
    a.nslices = 0; a.slice_counts = nullptr; a.slice_notes = nullptr;
    const size_t need = sample_restricted_workspace_bytes(rows, V);
    if (need > 0 && workspace != nullptr && (reinterpret_cast<uintptr_t>(workspace) & 15u) == 0 && workspace_bytes >= need) {
        a.nslices = slices_of(rows, V);
        a.slice_counts = static_cast<uint16_t*>(workspace);
        a.slice_notes = reinterpret_cast<SliceNotes*>(a.slice_counts + (size_t)rows * a.nslices * kArray);
        hipLaunchKernelGGL(count_slices_kernel, dim3((unsigned)(rows * a.nslices)), dim3(kSliceThreads), 0, stream, a);
        const hipError_t err = hipGetLastError();
        if (err != hipSuccess) return err;
        hipLaunchKernelGGL((sample_restricted_kernel<512, true>), dim3((unsigned)rows), dim3(512), 0, stream, a);
    } else if (rows <= compute_units() && V >= kFewWide) {
        hipLaunchKernelGGL((sample_restricted_kernel<1024, false>), dim3((unsigned)rows), dim3(1024), 0, stream, a);
    } else {
        hipLaunchKernelGGL((sample_restricted_kernel<512, false>), dim3((unsigned)rows), dim3(512), 0, stream, a);
    }
    return hipGetLastError();
}

}  // namespace e3
