// Structures shared by the host runtime and the gfx950 kernels of the TKdV
// rejection sampler.  Plain data only; no HIP types in the structs.
#pragma once

#include <stdint.h>

#include "../../include/tkdv.h"

namespace tkdv {

constexpr int kWave = 64;          // CDNA wavefront
constexpr int kTile = 32;          // proposals per wave tile (two lanes per proposal)
constexpr int kBlock = 256;        // threads per workgroup of the sampling kernels
// Workgroup of the default decision kernel of each K: at K <= 32 the
// half-period k_decide; at K = 64 and K = 128 the quarter-period kernel
// (tkdv_quarter.hip): workgroups of 256 threads at K = 64 (32 KB of tables
// with BF16x3, several workgroups per CU), of 768 at K = 128 (128 KB of
// tables, one workgroup of 12 waves per CU, 3 per SIMD).
constexpr int decide_block(int K) { return K == 128 ? 768 : kBlock; }
// The half-period k_decide at K = 64 (a tile variant of the sweep's tuner):
// one copy of its 64 KB of tables served 12 waves, 3 per SIMD (168 registers a
// lane; four waves spill inside the tile loop).
constexpr int kHalfPeriod64Block = 768;
constexpr int kSynthBlock = 512;   // threads per workgroup of the standalone synthesis kernel
constexpr int kClaimTiles = 64;    // most tiles of a work-queue claim (2048 proposals);
                                   // lane c keeps the accept word of tile c
// Accepted-count sampling of one point or a batch decides at least this many
// tiles (2^21 proposals, divided among the points), target met or not.
constexpr uint64_t kAlwaysTiles = 1ull << 16;
// Tiles of a point's range of n tiles that are dealt out evenly to the waves
// instead of claimed (one of n_points points in the call).  The claims of one
// queue serialise on its counter, about 20 ns each: guided claims down to two
// tiles took 0.64 ms for a million proposals at K = 8, claims of a fixed 64 tiles
// 0.22 ms with 489 waves busy, even shares 0.15 ms (decisions 90 -> 30 us); and
// 2e7 proposals at K = 16 with FP32 products 0.94 ms claimed, 0.82 ms dealt out.
// But the waves of a SIMD advance at different speeds (the oldest first), so
// that a long even share leaves the youngest alone at its end: a billion
// proposals at K = 32 took 50.2 ms claimed, 52.3 ms with half and 56.6 ms with
// 7/8 of them dealt out.  So ranges up to 2^20 tiles per call are dealt out
// and larger ones claimed.  at_least: tiles wanted in any case (accepted-count
// mode, where the rest of the range may not be needed).
constexpr uint64_t kMaxStatic = 1ull << 20;
// A launch whose tiles are all dealt out takes up to kDealtRounds rounds of
// workgroups, of waves with kDealtTiles tiles each at least: the next workgroup
// starts where one ends, which evens out the waves' different speeds (K = 32, 3e7
// proposals: 1.59 -> 1.47 ms; K = 64: 3.40 -> 3.14; K = 8: 517 -> 479 us; 1e6 and
// fewer are one round).  Larger ranges dealt out in 16 or 64 rounds are no faster
// than claimed at K = 32 and slower at K = 64 and 128 (6e7 each: 41.0 -> 45.1 ms).
constexpr int kDealtRounds = 4, kDealtTiles = 16;
constexpr unsigned long long dealt_rounds(unsigned long long tiles, unsigned long long waves)
{
    const unsigned long long r = tiles / (waves * kDealtTiles);
    return r < 1 ? 1 : (r > kDealtRounds ? kDealtRounds : r);
}
constexpr uint64_t static_share(uint64_t n, uint64_t at_least, int n_points)
{
    const uint64_t cap = kMaxStatic / (uint64_t)n_points;
    if (at_least >= n) return n <= cap ? n : 0;
    return at_least < cap ? at_least : cap;
}
// The ordered output finds the accepted sample of a rank through the accept counts
// of segments of 8 to 2048 words (a power of two, the same for all points of a
// call): about kSegments of them, as many as waves to count them, unless they would
// be longer than 2048 words.
constexpr int kSegWordsMax = 2048, kSegments = 4096;
// log2 of a segment's words for a call of `words` accept words
constexpr int seg_shift_for(unsigned long long words)
{
    int sh = 3;
    while ((1 << sh) < kSegWordsMax && words > ((unsigned long long)kSegments << sh)) ++sh;
    return sh;
}
// most segments of a call of n_points points with at most `words` accept words
constexpr unsigned long long max_segments(unsigned long long words, int n_points)
{
    const unsigned long long by_size = words / kSegWordsMax;
    return (by_size > (unsigned long long)kSegments ? by_size : (unsigned long long)kSegments) +
           (unsigned long long)n_points;
}
// The accepted samples that a point's output takes are cut into runs of R = 2^j
// successive ranks, one wave each, whose statistics are summed in the order of the
// runs.  R follows from the number of samples (and K) alone, so that the moments are
// a function of the samples: not of the tiles decided past a target, whose number
// depends on timing, nor of the call's other points.  Runs shorter than a tile of the
// ordered output (32 proposals, 16 at K = 64 and 128) leave lanes idle, but a wave
// reads the accept words between its samples one group after the other (some 800 samples
// of 1e9 proposals at K = 16: 91 us in runs of 16, 50 in runs of 8); they are for few
// samples, of which many points still fit the chip.  From there on short runs share
// out one point's samples better (3e4 at K = 64: 31 us in runs of 32, 51 in runs of
// 64), long ones take less to find their first sample (24 points of 1e5 at K = 16: 199
// us in runs of 64, 173 in runs of 128) and give the final sums, which one workgroup a
// point reads, fewer records.
constexpr unsigned long long run_most(int K, int j)  // most samples that are cut into runs of 2^j
{
    constexpr unsigned long long few[2][9] = {
        {64, 128, 256, 4096, 8192, 32768, 65536, 1 << 19, 1 << 21},   // K <= 32
        {64, 128, 256, 2048, 8192, 65536, 1 << 19, 1 << 20, 1 << 21}};  // K >= 64: workgroups of 8 waves, dear tiles
    return j < 9 ? few[K >= 64][j] : 32ull << (2 * j);
}
constexpr int run_shift(int K, unsigned long long samples)
{
    int j = 0;
#pragma unroll 1
    while (j < 28 && samples > run_most(K, j)) ++j;
    return j;
}
constexpr unsigned long long runs_of(int K, unsigned long long samples)
{
    const int j = run_shift(K, samples);
    return (samples >> j) + ((samples & ((1ull << j) - 1)) != 0);
}
// most runs of a point with at most `samples` samples: those of the most samples
// with the next shorter runs, if these are more
constexpr unsigned long long max_runs(int K, unsigned long long samples)
{
    const int j = run_shift(K, samples);
    const unsigned long long own = runs_of(K, samples), shorter = j > 0 ? run_most(K, j - 1) >> (j - 1) : 0ull;
    return own > shorter ? own : shorter;
}
constexpr int kNBins = TKDV_NBINS;
constexpr int kMixBlock = 1024;    // threads per workgroup of the mixture sampling kernel
constexpr int kMixS = TKDV_MIX_S;  // xi-shifts of the learned mixture

// Per-point constants, laid out for wave-uniform (scalar) loads; sig is also
// read four floats at a time per lane (K = 128 kernels).
struct alignas(16) DevPoint {
    float sig[TKDV_KMAX];    // proposal standard deviations s_k (1 for the uniform proposal)
    double sig64[TKDV_KMAX]; // the same in FP64 (sqrt of the plan's s_k^2)
    // FP32 fast path: log a = neg_bp_K2 * t + c3coef * S3 + Kf * log1p(g_coef * t) - log_M
    float neg_bp_K2;         // -beta'/K^2
    float c3coef;            // beta' c/(E0 K^2) * (pi/(3N)) * (2 E0/pi)^{3/2}
    float g_coef;            // alpha* beta'/K^3   (Sigma proposal; 0 for uniform)
    float Kf;                // K                  (Sigma proposal; 0 for uniform)
    float log_M;             // log M rounded to FP32
    float tau;               // decision window: |log U - log a| < tau -> FP64 re-decision
    float e_lo, e_hi;        // exp(-tau), exp(tau): the window in terms of U and a
    int32_t K;
    int32_t proposal;
    uint32_t point_id;
    uint32_t key0, key1;     // Philox key = seed
    uint32_t pad0;
    // FP64 re-decision
    double E0, beta_p, c32, alpha_star, log_M64;
    double amp;              // sqrt(2 E0/pi)
    // work description
    uint64_t i0;             // first proposal index
    uint64_t n;              // proposals to cover (upper bound in accepted-count mode)
    uint64_t n_tiles;        // ceil(n / 32)
    uint64_t target;         // accepted-sample target (UINT64_MAX in proposal-count mode)
    uint64_t static_tiles;   // the first tiles, dealt out evenly to the waves (static_share)
    uint64_t bm_off;         // first bitmap word of this point
    uint64_t out_off;        // first output row of this point
    uint64_t capacity;       // output rows available to this point
    uint64_t row_stride;     // floats between consecutive output rows
};

// Per-point constants of the learned mixture proposal (see tkdv_mixture).
// Its tables live at tab_off in the mixture table buffer:
//   y tables  B[(q, j)][c] = a_c (R_j V C^T)_{c q} as matrix-core A operands,
//             row tile q (rank index), row j (shift) -- BF16 hi, BF16 lo, FP32;
//             C is the upper Cholesky factor of (I + V^T D^-1 V)^-1 = C^T C, so
//             the products give z_j = C y_j and y_j^T G^-1 y_j = |z_j|^2;
//   RV table  (R_j V)_c for shift j, half h, coordinate k of that half:
//             float2 at ((2 j + h) (2K + 2) + 2 k) floats (rows padded by
//             two floats to spread the shifts over the LDS banks).
struct DevMix {
    float sqd[TKDV_KMAX];    // sqrt(d_k)
    float a[TKDV_KMAX];      // 1/d_k
    float c_net;             // ln(1 - eps) - ln|L0|/2 - ln S
    float c_g;               // ln eps + sum_k ln(1 + alpha beta' k^2/K^3)
    float invB;              // 1/B rounded to FP32
    uint32_t E, B;           // component word: w < E -> g_Sigma, else j = (w - E) div B
    // FP64 re-decision
    double a64[TKDV_KMAX], sqd64[TKDV_KMAX];
    double V64[2 * TKDV_KMAX][TKDV_MIX_R];
    double gi64[TKDV_MIX_R][TKDV_MIX_R];
    double cs64[kMixS], sn64[kMixS];  // cos, sin of 2 pi m/S
    double logdetL0, lng, log_eps, log_1m_eps;
    uint64_t tab_off;        // bytes
    uint64_t pad;
};

template <int K>
constexpr int mix_ytab_bf16_bytes() { return 2 * (K / 8) * kWave * 16; }
template <int K>
constexpr int mix_ytab_f32_bytes() { return 2 * (K / 4) * kWave * 16; }
template <int K>
constexpr int mix_rv_bytes() { return kMixS * 2 * (2 * K + 2) * 4; }
// per point: y hi, y lo, y f32, RV
template <int K>
constexpr int mix_point_bytes()
{
    return 2 * mix_ytab_bf16_bytes<K>() + mix_ytab_f32_bytes<K>() + mix_rv_bytes<K>();
}

// Device-side counters per point (zeroed before every launch sequence).  Updates
// of one line by all waves serialise (10 to 20 ns each on a memory that eight
// dies share), and in small calls all waves report at once; so what waves report
// is spread over kShards lines, workgroup b using line b mod kShards (the
// decisions of 2e6 proposals at K = 16 where nearly all are accepted: 0.31 ms
// with one line, 0.18 ms with eight).
constexpr int kShards = 8;
struct alignas(128) CounterShard {
    unsigned long long accepted;      // accepted-count mode: definite accepts of the finished tiles
    unsigned long long finished;      // accepted-count mode: finished tiles
    unsigned long long violations;    // proposals with log a > 0
    unsigned long long deferred;      // proposals sent to the FP64 re-decision
    unsigned int max_log_a_key;       // order-preserving encoding of the largest log a
    unsigned int pad;
};
struct alignas(128) DevCounters {
    unsigned long long next_tile;     // work-queue head (tiles claimed after the static ones)
    unsigned long long pad0[15];      // a line of its own: every claim goes through it
    unsigned long long last_index;    // accepted-count mode: index of the target-th sample
    unsigned long long pad1[15];
    CounterShard shard[kShards];
};
// the sums over the shards
constexpr CounterShard shard_totals(const DevCounters &c)
{
    CounterShard t = c.shard[0];
    for (int s = 1; s < kShards; ++s) {
        t.accepted += c.shard[s].accepted;
        t.finished += c.shard[s].finished;
        t.violations += c.shard[s].violations;
        t.deferred += c.shard[s].deferred;
        t.max_log_a_key = c.shard[s].max_log_a_key > t.max_log_a_key ? c.shard[s].max_log_a_key : t.max_log_a_key;
    }
    return t;
}

// Where a point's accepted samples are (k_seg_scan).
struct PointRanks {
    unsigned long long samples;            // those that its output takes
    unsigned long long seg_first, n_segs;  // its segments, of 2^seg_shift words
    unsigned long long base;               // accepted before them (all points')
    unsigned long long n_words;            // its accept words
    int seg_shift, pad;
};

// Statistics of a run of ranks (FP64 sums in the order of the ranks).
struct RunStats {
    double S1, S2, S3, S4;
    unsigned long long peak_index;  // proposal index of the sample with the largest grid value
    unsigned int peak_key;          // float_key of that value of u~ (0: no sample)
    unsigned int n_exceed;          // grid values above 2 sigma
    unsigned int n_exceed4;         // grid values above 4 sigma
    unsigned int n_max4;            // samples whose largest grid value is above 4 sigma
};

// Per-point result of the finalisation kernel.
struct PointResult {
    double S1, S2, S3, S4;
    unsigned long long n_exceed;
    unsigned long long n_exceed4, n_max4, peak_index;  // as in RunStats
    unsigned int peak_key, pad;
    unsigned long long n_samples;      // accepted samples covered by the statistics
    unsigned long long n_accepted;     // all accepted in the processed range
    unsigned long long n_written;
    unsigned long long n_processed;    // proposals whose decision exists
    unsigned long long hist[kNBins];
};

// Per-point state of a windowed sweep (accepted-count sampling in windows of
// proposals; the device advances it after every window).
struct SweepState {
    uint64_t i_start, i_end;      // proposal indices [i_start, i_end) of the point
    uint64_t window;              // proposals of the first window (of every window when not adaptive)
    uint64_t target;              // accepted samples wanted
    uint64_t capacity, out_off;   // output rows of the point
    uint64_t accepted;            // accepted samples so far (at most target)
    uint64_t written;             // rows written so far
    uint64_t n_proposed;          // proposals consumed (up to the target-th sample)
    uint64_t n_fixups, n_violations;
    uint32_t done, max_log_a_key;
    PointResult total;            // statistics of the accepted samples so far
};

// Cuts of every point's words or ranks into pieces: the first piece of each point
// and, from bit kCutShiftBit on, log2 of its pieces' length; then their number.
constexpr int kCutShiftBit = 48;
struct Cuts {
    unsigned long long at[1];
};
constexpr size_t cuts_bytes(int n_points) { return sizeof(Cuts) + sizeof(unsigned long long) * (size_t)n_points; }

// Shared state of a sweep on the device.
struct SweepGlobal {
    unsigned long long pool_tiles;   // accept-bitmap words available to one window
    unsigned long long active;       // points not done
    unsigned long long windows;      // windows run with at least one point active
    unsigned long long overflow;     // a window's FP64 re-decision list overflowed
    unsigned long long defer_cap;
    int adaptive;                    // 1: size each window from the measured acceptance
    int pad;
};

struct KernelArgs {
    const DevPoint *pts;
    int n_points;
    int blocks_per_cu;     // decide-kernel workgroups per compute unit (0: as many as fit)
    int dealt;             // every tile of the launch is dealt out (static_share): rounds of workgroups
    DevCounters *cnt;
    uint32_t *bitmap;
    unsigned long long *defer_list;
    unsigned long long *defer_count;
    unsigned long long defer_cap;
    const void *phi_hi;    // BF16 fragment table (hi), or FP32 fragment table
    const void *phi_lo;    // BF16 fragment table (lo)
    const DevMix *mix;     // per point (learned proposal only)
    const char *mix_tab;   // mixture tables (learned proposal only)
    // optional per-proposal outputs of the evaluation entry point (point 0 only)
    float *dbg_xhat, *dbg_t, *dbg_s3, *dbg_log_a, *dbg_log_u;
    // sweeps: the number of unfinished points (NULL elsewhere)
    const unsigned long long *d_active;
    // ordered output: the segments of the accept words, their accept counts and
    // exclusive prefix (over all points, and the sum), where each point's samples are,
    // the runs of ranks, their statistics, and the u(0) histograms [point][kShards][kNBins]
    Cuts *seg;
    unsigned int *seg_cnt;
    unsigned long long *seg_base;
    PointRanks *ranks;
    Cuts *runs;
    RunStats *run_stats;
    unsigned long long *hist;
    PointResult *res;
};

}  // namespace tkdv
