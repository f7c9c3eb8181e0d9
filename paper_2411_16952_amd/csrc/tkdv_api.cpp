// C ABI of the gfx950 TKdV rejection sampler: context, workspaces, synthesis
// tables, argument checking and the launch sequence of one sampling call.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

#include "../../include/tkdv.h"
#include "tkdv_extremes.h"
#include "tkdv_internal.h"
#include "tkdv_kernels.h"
#include "tkdv_host_math.h"
#include "tkdv_mixture.h"
#include "tkdv_plan.h"
#include "tkdv_plan_gpu.h"
#include "tkdv_runtime.h"
#include "tkdv_scratch.h"
#include "tkdv_sir.h"

using namespace tkdv;

namespace {

const double kPi = 3.14159265358979323846;

// Plain BF16 products miss the 1e-3 tolerance on H3 in the worst case, so no
// accept decision is taken with them; the synthesis alone still offers them.
const char *const kBf16Refused =
    "plain BF16 synthesis is not used for decisions: its worst-case H3 error exceeds 1e-3 of the "
    "cube-sum scale (use TKDV_BF16X3 or TKDV_FP32)";

struct DevBuf {
    void *p = nullptr;
    size_t bytes = 0;
};

std::mutex g_err_mu;
std::string g_last_error;  // for calls without a context

// The GPU path's mode counts: K = 8 << ki for ki < kNumK.
constexpr int kNumK = 5;
int kindex(int K)
{
    switch (K) {
    case 8: return 0;
    case 16: return 1;
    case 32: return 2;
    case 64: return 3;
    case 128: return 4;
    default: return -1;
    }
}

}  // namespace

struct tkdv_ctx {
    int device = 0;
    int n_cu = 0;
    std::string last_error;
    DevBuf bitmap, defer_list, state, points, seg, seg_cnt, seg_base, ranks, runs, run_stats;  // state: CallState, points: PointList
    DevBuf mix, mix_tab;  // learned-proposal constants and tables of the current call
    // K = 128 (index 4): the quarter-period tables of k_decide128 (BF16 hi, lo, FP32)
    DevBuf phi_hi[kNumK], phi_lo[kNumK], phi_f32[kNumK];
    DevBuf q64_hi, q64_lo, q64_f32;  // K = 64's quarter-period decision tables
    DevBuf qstat[2];                 // quarter-period statistics tables, K = 64 and 128
    // the same tables with the odd-mode rows scaled by sqrt(3), for the kernels
    // that form S3 in the half-period form (K >= 16): s3_tables()
    DevBuf phi3_hi[kNumK], phi3_lo[kNumK], phi3_f32[kNumK];
    void *h_state = nullptr;  // pinned: CallState up to the histograms
    size_t h_state_bytes = 0;
    void *h_points = nullptr;  // pinned: PointList
    size_t h_points_bytes = 0;
    void *h_misc = nullptr;  // pinned: tkdv_extremes
    size_t h_misc_bytes = 0;
    hipEvent_t ev[6] = {};  // phase boundaries of the last call
    tkdv_timing timing = {};
    // sweep: launch configuration per (K index, precision), its own stream
    // (captured into graphs) joined to the caller's stream by events
    tkdv_launch_cfg lcfg[kNumK][3];
    hipStream_t sweep_stream = nullptr;
    hipEvent_t join[2] = {};
    DevBuf sweep, active;
    DevBuf plan_pts, plan_val, plan_x, plan_ev, plan_mix, plan_user;  // tkdv_plan_batch, _mixture_batch
    DevBuf ext_keys, ext_jmax, ext_misc;  // tkdv_extremes
    DevBuf sir_pt, sir_w, sir_tile, sir_chunk, sir_part;  // tkdv_sir
    void *h_poll = nullptr;  // pinned: active count, FP64 list count
    std::string arch;
    int mv_policy = TKDV_MV_RAISE;  // what a proposal with f/(M g) > 1 triggers
};

namespace {

tkdv_status set_err(tkdv_ctx *ctx, tkdv_status st, const std::string &msg)
{
    if (ctx) ctx->last_error = msg;
    std::lock_guard<std::mutex> g(g_err_mu);
    g_last_error = msg;
    return st;
}

#define HIP_TRY(ctx, expr)                                                                             \
    do {                                                                                               \
        hipError_t _e = (expr);                                                                        \
        if (_e != hipSuccess)                                                                          \
            return set_err((ctx), TKDV_E_DEVICE, std::string(#expr) + ": " + hipGetErrorString(_e)); \
    } while (0)

hipError_t ensure(DevBuf &b, size_t bytes)
{
    if (b.bytes >= bytes && b.p) return hipSuccess;
    if (b.p) {
        hipError_t e = hipFree(b.p);
        if (e != hipSuccess) return e;
        b.p = nullptr;
        b.bytes = 0;
    }
    size_t want = std::max<size_t>(bytes, 256);
    hipError_t e = hipMalloc(&b.p, want);
    if (e != hipSuccess) return e;
    b.bytes = want;
    return hipSuccess;
}

hipError_t ensure_host(void *&p, size_t &have, size_t bytes)
{
    if (have >= bytes && p) return hipSuccess;
    if (p) {
        hipError_t e = hipHostFree(p);
        if (e != hipSuccess) return e;
        p = nullptr;
        have = 0;
    }
    size_t want = std::max<size_t>(bytes, 4096);
    hipError_t e = hipHostMalloc(&p, want, hipHostMallocDefault);
    if (e != hipSuccess) return e;
    have = want;
    return hipSuccess;
}

// Quarter-period tables (tkdv_quarter.hip), K = 64 and 128, N = 4K.
//   Decision tables on the representatives xi_rho = pi (2 rho + 1)/N, rho < K
//   (the grid offset by half a step, points in (0, pi/2)): for tile tau
//   (rho = 16 tau + l % 16), output o (0: cos, even
//   modes; 1: cos, odd modes; 2: sin, even; 3: sin, odd; o > 0 scaled by
//   sqrt 3) and lane group g = l/16, the entry of mode
//   k = 32 g + 2 idx + (o even ? 2 : 1), where idx = 8 r + e in the BF16
//   layout [tau][o][r < 2][64 lanes][e < 8] (hi, lo) and idx = 4 q + e in the
//   FP32 layout [tau][o][q < 4][64 lanes][e < 4].
//   Statistics tables (FP32): the same layout on the statistics grid's own
//   representatives xi_rho = 2 pi rho/N, rho < K, unscaled.
//   Angles are reduced exactly in integers before the FP64 cos/sin.
hipError_t upload_quarter(int K, DevBuf &d_hi, DevBuf &d_lo, DevBuf &d_f32)
{
    const int N = 4 * K, CPL = K / 4, TILES = K / 16, STEPS = K / 64, QG = K / 32;
    const double r3 = std::sqrt(3.0);
    // entry of output o at representative rho for mode k: angle k pi (2 rho + 1)/N
    auto qval = [&](int o, int k, int rho) {
        const long m = ((long)k * (2 * rho + 1)) % (2 * N);
        const double ang = kPi * (double)m / N;
        const double v = (o < 2) ? std::cos(ang) : std::sin(ang);
        return o == 0 ? v : r3 * v;
    };
    auto mode = [&](int o, int g, int idx) { return CPL * g + 2 * idx + ((o == 0 || o == 2) ? 2 : 1); };
    std::vector<uint16_t> hi((size_t)TILES * 4 * STEPS * 64 * 8), lo(hi.size());
    for (int tau = 0; tau < TILES; ++tau)
        for (int o = 0; o < 4; ++o)
            for (int r = 0; r < STEPS; ++r)
                for (int l = 0; l < 64; ++l)
                    for (int e = 0; e < 8; ++e) {
                        const double v = qval(o, mode(o, l / 16, 8 * r + e), 16 * tau + l % 16);
                        const uint16_t h = bf16_bits((float)v);
                        const size_t idx = ((((size_t)tau * 4 + o) * STEPS + r) * 64 + l) * 8 + e;
                        hi[idx] = h;
                        lo[idx] = bf16_bits((float)(v - (double)bf16_value(h)));
                    }
    std::vector<float> f32((size_t)TILES * 4 * QG * 64 * 4);
    for (int tau = 0; tau < TILES; ++tau)
        for (int o = 0; o < 4; ++o)
            for (int q = 0; q < QG; ++q)
                for (int l = 0; l < 64; ++l)
                    for (int e = 0; e < 4; ++e)
                        f32[((((size_t)tau * 4 + o) * QG + q) * 64 + l) * 4 + e] =
                            (float)qval(o, mode(o, l / 16, 4 * q + e), 16 * tau + l % 16);
    hipError_t e = ensure(d_hi, hi.size() * 2);
    if (e == hipSuccess) e = ensure(d_lo, lo.size() * 2);
    if (e == hipSuccess) e = ensure(d_f32, f32.size() * 4);
    if (e == hipSuccess) e = hipMemcpy(d_hi.p, hi.data(), hi.size() * 2, hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemcpy(d_lo.p, lo.data(), lo.size() * 2, hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemcpy(d_f32.p, f32.data(), f32.size() * 4, hipMemcpyHostToDevice);
    return e;
}

hipError_t upload_quarter_stats(int K, DevBuf &d_f32)
{
    const int N = 4 * K, CPL = K / 4, TILES = K / 16, QG = K / 32;
    auto mode = [&](int o, int g, int idx) { return CPL * g + 2 * idx + ((o == 0 || o == 2) ? 2 : 1); };
    std::vector<float> f32((size_t)TILES * 4 * QG * 64 * 4);
    for (int tau = 0; tau < TILES; ++tau)
        for (int o = 0; o < 4; ++o)
            for (int q = 0; q < QG; ++q)
                for (int l = 0; l < 64; ++l)
                    for (int e = 0; e < 4; ++e) {
                        const int k = mode(o, l / 16, 4 * q + e), rho = 16 * tau + l % 16;
                        const double ang = 2.0 * kPi * (double)(((long)k * rho) % N) / N;
                        f32[((((size_t)tau * 4 + o) * QG + q) * 64 + l) * 4 + e] =
                            (float)(o < 2 ? std::cos(ang) : std::sin(ang));
                    }
    hipError_t e = ensure(d_f32, f32.size() * 4);
    if (e == hipSuccess) e = hipMemcpy(d_f32.p, f32.data(), f32.size() * 4, hipMemcpyHostToDevice);
    return e;
}

tkdv_status build_tables128(tkdv_ctx *ctx)
{
    HIP_TRY(ctx, upload_quarter(128, ctx->phi_hi[4], ctx->phi_lo[4], ctx->phi_f32[4]));
    HIP_TRY(ctx, upload_quarter_stats(128, ctx->qstat[1]));
    return TKDV_OK;
}

// Synthesis tables for K modes on the grid xi_j = -pi + 2 pi j/N, N = 4K.
// Row (block b, mode k) of Phi is cos(k xi_j) (b = 0) or sin(k xi_j) (b = 1);
// angles are reduced exactly: k xi_j = -k pi + 2 pi (k j mod N)/N.  For
// K >= 16 a second set carries the odd-mode rows times sqrt(3): the half-period
// cube sum 2 E (E^2 + 3 O^2) then reads 2 E (E^2 + o^2) with o = sqrt(3) O.
tkdv_status build_tables(tkdv_ctx *ctx, int K)
{
    const int ki = kindex(K);
    if (ctx->phi_hi[ki].p) return TKDV_OK;
    const int N = 4 * K, T = K / 8, S = K / 8, Q = K / 4;
    auto phi = [&](int block, int k, int j) {
        const long r = ((long)k * j) % N;
        const double ang = 2.0 * kPi * (double)r / N;
        const double sign = (k & 1) ? -1.0 : 1.0;  // shift by -k pi
        return block == 0 ? sign * std::cos(ang) : sign * std::sin(ang);
    };
    auto upload = [&](double odd_scale, DevBuf &d_hi, DevBuf &d_lo, DevBuf &d_f32) -> hipError_t {
        auto row = [&](int block, int k, int j) { return ((k & 1) ? odd_scale : 1.0) * phi(block, k, j); };
        std::vector<uint16_t> hi((size_t)T * S * 64 * 8), lo(hi.size());
        for (int t = 0; t < T; ++t)
            for (int s = 0; s < S; ++s)
                for (int l = 0; l < 64; ++l)
                    for (int e = 0; e < 8; ++e) {
                        const int block = l / 32, j = 32 * t + l % 32, k = 8 * s + e + 1;
                        const double v = row(block, k, j);
                        const uint16_t h = bf16_bits((float)v);
                        const double rem = v - (double)bf16_value(h);
                        const size_t idx = (((size_t)t * S + s) * 64 + l) * 8 + e;
                        hi[idx] = h;
                        lo[idx] = bf16_bits((float)rem);
                    }
        std::vector<float> f32((size_t)T * Q * 64 * 4);
        for (int t = 0; t < T; ++t)
            for (int q = 0; q < Q; ++q)
                for (int l = 0; l < 64; ++l)
                    for (int e = 0; e < 4; ++e) {
                        const int block = l / 32, j = 32 * t + l % 32, k = 4 * q + e + 1;
                        f32[(((size_t)t * Q + q) * 64 + l) * 4 + e] = (float)row(block, k, j);
                    }
        hipError_t e = ensure(d_hi, hi.size() * 2);
        if (e == hipSuccess) e = ensure(d_lo, lo.size() * 2);
        if (e == hipSuccess) e = ensure(d_f32, f32.size() * 4);
        if (e == hipSuccess) e = hipMemcpy(d_hi.p, hi.data(), hi.size() * 2, hipMemcpyHostToDevice);
        if (e == hipSuccess) e = hipMemcpy(d_lo.p, lo.data(), lo.size() * 2, hipMemcpyHostToDevice);
        if (e == hipSuccess) e = hipMemcpy(d_f32.p, f32.data(), f32.size() * 4, hipMemcpyHostToDevice);
        return e;
    };
    if (K == 128) return build_tables128(ctx);
    if (K == 64) {
        HIP_TRY(ctx, upload_quarter(64, ctx->q64_hi, ctx->q64_lo, ctx->q64_f32));
        HIP_TRY(ctx, upload_quarter_stats(64, ctx->qstat[0]));
    }
    if (K >= 16) HIP_TRY(ctx, upload(std::sqrt(3.0), ctx->phi3_hi[ki], ctx->phi3_lo[ki], ctx->phi3_f32[ki]));
    HIP_TRY(ctx, upload(1.0, ctx->phi_hi[ki], ctx->phi_lo[ki], ctx->phi_f32[ki]));
    return TKDV_OK;
}

// Tables read by the S3 kernels (k_decide, k_decide_mix, k_synth): the scaled
// set in the half-period form (16 <= K <= 64), the plain tables at K = 8, the
// quarter-period tables at K = 128.
// Tables of the default decision kernel of K = 8 << ki (variant 0 of the
// tuner's tile variants; the others read the S3 tables): the quarter-period
// tables at K = 64.
void s3_tables(const tkdv_ctx *ctx, int ki, int precision, const void *&hi, const void *&lo);
void decide_tables(const tkdv_ctx *ctx, int ki, int precision, int variant, const void *&hi, const void *&lo)
{
    if (ki == 3 && variant == 0) {
        hi = precision == TKDV_FP32 ? ctx->q64_f32.p : ctx->q64_hi.p;
        lo = ctx->q64_lo.p;
        return;
    }
    s3_tables(ctx, ki, precision, hi, lo);
}

void s3_tables(const tkdv_ctx *ctx, int ki, int precision, const void *&hi, const void *&lo)
{
    if (ki == 4) {  // K = 128: the quarter-period tables
        hi = precision == TKDV_FP32 ? ctx->phi_f32[4].p : ctx->phi_hi[4].p;
        lo = ctx->phi_lo[4].p;
        return;
    }
    const bool eo = ki >= 1;
    const DevBuf &h = precision == TKDV_FP32 ? (eo ? ctx->phi3_f32[ki] : ctx->phi_f32[ki])
                                             : (eo ? ctx->phi3_hi[ki] : ctx->phi_hi[ki]);
    hi = h.p;
    lo = eo ? ctx->phi3_lo[ki].p : ctx->phi_lo[ki].p;
}

tkdv_status check_point(tkdv_ctx *ctx, const tkdv_point &pt)
{
    if (pt.K < 1 || pt.K > TKDV_KMAX) return set_err(ctx, TKDV_E_ARG, "K out of range");
    if (kindex(pt.K) < 0) return set_err(ctx, TKDV_E_UNSUPPORTED, "GPU path supports K in {8,16,32,64,128}");
    if (!std::isfinite(pt.E0) || !(pt.E0 > 0.0)) return set_err(ctx, TKDV_E_ARG, "E0 must be finite and > 0");
    if (!std::isfinite(pt.beta_p) || pt.beta_p < 0.0)
        return set_err(ctx, TKDV_E_ARG, "beta' must be finite and >= 0");
    if (!std::isfinite(pt.c32)) return set_err(ctx, TKDV_E_ARG, "C3/C2 must be finite");
    return TKDV_OK;
}

// Upper bound on |log a_fast - log a_exact| (times 2) for the FP32 fast path:
//   max_j |du~_j| <= sqrt(K) (eps_synth + eps_x)  (Cauchy-Schwarz, |x^| = 1,
//   sum_k Phi_kj^2 = K), |dH3| <= E0 amp max|du~| + sum-of-cubes rounding
//   (sum_j u_j^2 = N E0/pi), the t terms carry 4 eps_x relative error, and
//   FP32 rounding of the terms of log a and of log U is added explicitly.
double window(const tkdv_point &pt, int proposal, int precision, double alpha, double log_M, double extra = 0.0)
{
    const int K = pt.K, N = 4 * K;
    const double eps_x = 1e-5;  // bound on |x^_fast - x^_exact|_2 (normals + projection)
    // relative error of a synthesis sum of products, per sum of |products|:
    // FP32 accumulation of 2K terms (2^-23 per addition, allowing truncation);
    // BF16 products: both operands rounded (2^-9 each); BF16x3: with
    // x = x_hi + x_lo + d, |d| <= 2^-18 |x| (two roundings to 8 significant
    // bits), dropping lo*lo and d leaves at most 3 * 2^-18 per product
    double eps_s;
    switch (precision) {
    case TKDV_FP32: eps_s = 2.0 * K * 0x1p-23; break;
    case TKDV_BF16: eps_s = 1.01 * 0x1p-8 + 2.0 * K * 0x1p-23; break;
    default: eps_s = 3.02 * 0x1p-18 + 2.0 * K * 0x1p-23; break;
    }
    const double amp = std::sqrt(2.0 * pt.E0 / kPi);
    const double du = std::sqrt((double)K) * (eps_s + eps_x);  // max_j |du~_j|, u~ unscaled
    const double umax = std::sqrt((double)K);                   // |u~_j| <= sqrt(K)
    // S3 = sum_j u~_j^3 with sum_j u~_j^2 = N/2 exactly: first-order error
    // 3 (N/2) du, plus FP32 accumulation of N cubes, |S3| <= umax N/2.
    const double err_S3 = 3.0 * (N / 2.0) * du + N * 0x1p-23 * umax * (N / 2.0);
    const double c3coef = pt.beta_p * std::fabs(pt.c32) / (pt.E0 * K * K) * (kPi / (3.0 * N)) * amp * amp * amp;
    const double err_H3term = c3coef * err_S3;
    // t = sum k^2 s_k: |dt| <= 2 K^2 |x^| |dx^| plus rounding
    const double err_t = 4.0 * eps_x * K * K + 64.0 * K * K * 0x1p-24;
    const double slope = pt.beta_p / ((double)K * K) * (1.0 + (proposal != TKDV_PROP_UNIFORM ? alpha : 0.0));
    const double err_tterm = slope * err_t;
    // FP32 rounding of the terms of log a (each bounded in magnitude) and of log U
    const double mag = pt.beta_p + K * std::log1p(alpha * pt.beta_p / K) + std::fabs(log_M) +
                       c3coef * umax * (N / 2.0);
    const double err_round = 16.0 * 0x1p-24 * (mag + 30.0);
    return 2.0 * (err_H3term + err_tterm + err_round + extra) + 1e-6;
}

// The rejection bound f <= M g (Sec. IV.A) with M from a search: after a run
// that saw log a > 0, log M is raised above the largest log a seen -- its
// FP32 value plus half the decision window (which bounds that value's error)
// plus log(1 + kRaiseMargin) -- and the point is run again from its first
// proposal, at most kMaxRaises times (tkdv_violation_policy).
constexpr int kMaxRaises = 4;
constexpr double kRaiseMargin = 0.02;
double raised_log_M(double log_M, double max_log_a, double tau)
{
    return log_M + std::max(max_log_a, 0.0) + 0.5 * tau + std::log1p(kRaiseMargin);
}

tkdv_status violation_error(tkdv_ctx *ctx, int p, const tkdv_stats &st)
{
    return set_err(ctx, TKDV_E_M_VIOLATION,
                   "point " + std::to_string(p) + ": " + std::to_string(st.n_M_violations) +
                       " proposals with f/(M g) > 1 (largest log a " + std::to_string(st.max_log_a) + ")");
}

void set_window(DevPoint &d, double tau)
{
    d.tau = (float)tau;
    // rounded inwards so that the FP32 products stay inside the exact window
    d.e_lo = (float)std::exp(-tau) * (1.0f - 0x1p-22f);
    d.e_hi = (float)std::exp(tau) * (1.0f + 0x1p-22f);
}

// The mixture keeps the Sigma component (its standard deviations and alpha*).
void fill_devpoint(DevPoint &d, const tkdv_point &pt, const tkdv_plan &pl, int proposal, int precision)
{
    std::memset(&d, 0, sizeof(d));
    const int K = pt.K, N = 4 * K;
    const bool sig = proposal != TKDV_PROP_UNIFORM;
    for (int k = 0; k < TKDV_KMAX; ++k) {
        const double s2 = (k < K && sig) ? pl.sigma2[k] : 1.0;
        d.sig64[k] = std::sqrt(s2);
        d.sig[k] = (float)d.sig64[k];
    }
    const double amp = std::sqrt(2.0 * pt.E0 / kPi);
    d.neg_bp_K2 = (float)(-pt.beta_p / ((double)K * K));
    d.c3coef = (float)(pt.beta_p * pt.c32 / (pt.E0 * K * K) * (kPi / (3.0 * N)) * amp * amp * amp);
    d.g_coef = sig ? (float)(pl.alpha_star * pt.beta_p / ((double)K * K * K)) : 0.0f;
    d.Kf = sig ? (float)K : 0.0f;
    d.log_M = (float)pl.log_M;
    set_window(d, window(pt, proposal, precision, pl.alpha_star, pl.log_M));
    d.K = K;
    d.proposal = proposal;
    d.point_id = pt.point_id;
    d.key0 = (uint32_t)pt.seed;
    d.key1 = (uint32_t)(pt.seed >> 32);
    d.E0 = pt.E0;
    d.beta_p = pt.beta_p;
    d.c32 = pt.c32;
    d.alpha_star = pl.alpha_star;
    d.log_M64 = pl.log_M;
    d.amp = amp;
}

struct Call {
    std::vector<DevPoint> pts;
    std::vector<int> plist_off, plist_n;  // per K index
    std::vector<int> plist;               // concatenated point lists
    unsigned long long total_tiles = 0, max_segs = 0, max_runs = 0, bitmap_words = 0;
};

// What a call starts from zero, and, up to the histograms, brings back: one
// region, one fill and one copy (four and three of them kept a small call's
// stream waiting for its host for 25 us of 145).
struct CallState {
    size_t results = 0, counters, defer_count, hist, bytes;
    explicit CallState(int np)
    {
        auto place = [&](size_t &at, size_t n) {
            at = bytes;
            bytes = (bytes + n + 255) & ~(size_t)255;
        };
        bytes = 0;
        place(results, sizeof(PointResult) * np);
        place(counters, sizeof(DevCounters) * np);
        place(defer_count, sizeof(unsigned long long));
        place(hist, sizeof(unsigned long long) * kShards * kNBins * np);
    }
    size_t back() const { return defer_count + sizeof(unsigned long long); }
};
// A call's points and their lists per K, one copy.
struct PointList {
    size_t plist, bytes;
    PointList(int np, size_t n_list) : plist(sizeof(DevPoint) * np), bytes(plist + sizeof(int) * n_list) {}
};

// Device buffers of one launch sequence (from the context's growable buffers,
// or carved from a fixed scratch array by the no-allocation entry point).
struct Workspace {
    uint32_t *bitmap;
    unsigned long long *defer_list, defer_cap;
    char *state;   // CallState
    char *points;  // PointList
    Cuts *seg, *runs;
    unsigned int *seg_cnt;
    unsigned long long *seg_base;
    PointRanks *ranks;
    RunStats *run_stats;
};

void set_state(KernelArgs &a, char *state, const CallState &cs)
{
    a.res = reinterpret_cast<PointResult *>(state + cs.results);
    a.cnt = reinterpret_cast<DevCounters *>(state + cs.counters);
    a.defer_count = reinterpret_cast<unsigned long long *>(state + cs.defer_count);
    a.hist = reinterpret_cast<unsigned long long *>(state + cs.hist);
}

// Host view of one launch sequence: the points, their lists per K and the
// most segments and runs (plain arrays, so that a caller need not allocate).
struct CallView {
    const DevPoint *pts;
    int np;
    const int *plist;
    int plist_len;
    int plist_off[kNumK], plist_n[kNumK];
    unsigned long long max_segs, max_runs;
};

CallView view_of(const Call &call)
{
    CallView v;
    v.pts = call.pts.data();
    v.np = (int)call.pts.size();
    v.plist = call.plist.data();
    v.plist_len = (int)call.plist.size();
    for (int ki = 0; ki < kNumK; ++ki) {
        v.plist_off[ki] = call.plist_off[ki];
        v.plist_n[ki] = call.plist_n[ki];
    }
    v.max_segs = call.max_segs;
    v.max_runs = call.max_runs;
    return v;
}

// The launch sequence of one sampling call on stream st: decisions per K,
// FP64 re-decision, and (stats) segments, ordered output with statistics and
// the per-point reduction; then the per-point results and counters are
// copied to res_out / cnt_out (host arrays [np], may be NULL).  Uses the
// context's pinned staging buffers (large enough for v.np points) and the
// synthesis tables of every K in the call (built); allocates nothing.
tkdv_status launch_sequence(tkdv_ctx *ctx, const CallView &v, const Workspace &w, int precision, int proposal,
                            float *d_xhat, unsigned long long *d_index, hipStream_t st, PointResult *res_out,
                            DevCounters *cnt_out, unsigned long long *n_deferred_out, float *dbg_xhat,
                            float *dbg_t, float *dbg_s3, float *dbg_la, float *dbg_lu, bool stats)
{
    const int np = v.np;
    // The pinned staging buffers are reused by later calls, so the stream must
    // have consumed them before we return (we synchronise at the end).
    const CallState cs(np);
    const PointList pl(np, (size_t)v.plist_len);
    char *h_points = static_cast<char *>(ctx->h_points), *h_state = static_cast<char *>(ctx->h_state);
    std::memcpy(h_points, v.pts, sizeof(DevPoint) * np);
    std::memcpy(h_points + pl.plist, v.plist, sizeof(int) * v.plist_len);
    HIP_TRY(ctx, hipMemcpyAsync(w.points, h_points, pl.bytes, hipMemcpyHostToDevice, st));
    HIP_TRY(ctx, launch_fill_u32(w.state, cs.bytes / 4, 0u, st));

    KernelArgs a;
    std::memset(&a, 0, sizeof(a));
    a.seg = w.seg;
    a.seg_cnt = w.seg_cnt;
    a.seg_base = w.seg_base;
    a.ranks = w.ranks;
    a.runs = w.runs;
    a.run_stats = w.run_stats;
    set_state(a, w.state, cs);
    a.pts = reinterpret_cast<const DevPoint *>(w.points);
    a.n_points = np;
    a.bitmap = w.bitmap;
    a.defer_list = w.defer_list;
    a.defer_cap = w.defer_cap;
    a.dbg_xhat = dbg_xhat;
    a.dbg_t = dbg_t;
    a.dbg_s3 = dbg_s3;
    a.dbg_log_a = dbg_la;
    a.dbg_log_u = dbg_lu;
    if (proposal == TKDV_PROP_MIXTURE) {
        a.mix = reinterpret_cast<const DevMix *>(ctx->mix.p);
        a.mix_tab = reinterpret_cast<const char *>(ctx->mix_tab.p);
    }
    a.dealt = 1;
    for (int q = 0; q < np; ++q)
        if (v.pts[q].static_tiles < v.pts[q].n_tiles) a.dealt = 0;
    const int *d_plist = reinterpret_cast<const int *>(w.points + pl.plist);
    std::memset(&ctx->timing, 0, sizeof(ctx->timing));
    HIP_TRY(ctx, hipEventRecord(ctx->ev[0], st));
    for (int ki = 0; ki < kNumK; ++ki) {
        if (v.plist_n[ki] == 0) continue;
        const int K = 8 << ki;
        // the largest K of the call sets the reported workgroup size
        ctx->timing.decide_block = proposal == TKDV_PROP_MIXTURE ? kMixBlock : decide_block(K);
        decide_tables(ctx, ki, precision, 0, a.phi_hi, a.phi_lo);
        unsigned long long tiles = 0;
        for (int q = 0; q < v.plist_n[ki]; ++q) tiles += v.pts[v.plist[v.plist_off[ki] + q]].n_tiles;
        if (proposal == TKDV_PROP_MIXTURE)
            HIP_TRY(ctx, launch_decide_mix(K, precision, a, d_plist + v.plist_off[ki], v.plist_n[ki], ctx->n_cu,
                                           tiles, st, &ctx->timing.decide_grid));
        else
            HIP_TRY(ctx, launch_decide(K, precision, proposal, a, d_plist + v.plist_off[ki], v.plist_n[ki],
                                       ctx->n_cu, tiles, st, &ctx->timing.decide_grid));
        ctx->timing.decide_launches++;
    }
    HIP_TRY(ctx, hipEventRecord(ctx->ev[1], st));
    auto fixup = proposal == TKDV_PROP_MIXTURE ? launch_fixup_mix : launch_fixup;
    bool plan = stats;  // the first launch lays out the segments
    for (int ki = 0; ki < kNumK; ++ki) {
        if (v.plist_n[ki] == 0) continue;
        HIP_TRY(ctx, fixup(8 << ki, a, plan, ctx->n_cu, st));
        plan = false;
    }
    HIP_TRY(ctx, hipEventRecord(ctx->ev[2], st));
    if (stats) {
        HIP_TRY(ctx, launch_segments(a, v.max_segs, ctx->n_cu, st));
        HIP_TRY(ctx, hipEventRecord(ctx->ev[3], st));
        for (int ki = 0; ki < kNumK; ++ki) {
            if (v.plist_n[ki] == 0) continue;
            a.phi_hi = ki >= 3 ? ctx->qstat[ki - 3].p : ctx->phi_f32[ki].p;
            HIP_TRY(ctx, launch_materialize(8 << ki, proposal, a, v.max_runs, d_xhat, d_index, ctx->n_cu, st));
        }
        HIP_TRY(ctx, hipEventRecord(ctx->ev[4], st));
        HIP_TRY(ctx, launch_finalize(a, st));
        HIP_TRY(ctx, hipEventRecord(ctx->ev[5], st));
    }
    HIP_TRY(ctx, hipMemcpyAsync(h_state, w.state, cs.back(), hipMemcpyDeviceToHost, st));
    HIP_TRY(ctx, hipStreamSynchronize(st));
    {
        float ms = 0.0f;
        HIP_TRY(ctx, hipEventElapsedTime(&ms, ctx->ev[0], ctx->ev[1]));
        ctx->timing.decide_ms = ms;
        HIP_TRY(ctx, hipEventElapsedTime(&ms, ctx->ev[1], ctx->ev[2]));
        ctx->timing.fixup_ms = ms;
        if (stats) {
            HIP_TRY(ctx, hipEventElapsedTime(&ms, ctx->ev[2], ctx->ev[3]));
            ctx->timing.segments_ms = ms;
            HIP_TRY(ctx, hipEventElapsedTime(&ms, ctx->ev[3], ctx->ev[4]));
            ctx->timing.materialize_ms = ms;
            HIP_TRY(ctx, hipEventElapsedTime(&ms, ctx->ev[4], ctx->ev[5]));
            ctx->timing.finalize_ms = ms;
            HIP_TRY(ctx, hipEventElapsedTime(&ms, ctx->ev[0], ctx->ev[5]));
        } else {
            HIP_TRY(ctx, hipEventElapsedTime(&ms, ctx->ev[0], ctx->ev[2]));
        }
        ctx->timing.total_ms = ms;
    }
    const unsigned long long n_def = *reinterpret_cast<unsigned long long *>(h_state + cs.defer_count);
    if (n_deferred_out) *n_deferred_out = n_def;
    if (res_out && stats) std::memcpy(res_out, h_state + cs.results, sizeof(PointResult) * np);
    if (cnt_out) std::memcpy(cnt_out, h_state + cs.counters, sizeof(DevCounters) * np);
    if (n_def > w.defer_cap)
        return set_err(ctx, TKDV_E_CAPACITY, "FP64 re-decision list overflowed (" + std::to_string(n_def) + " > " +
                                                 std::to_string(w.defer_cap) + ")");
    return TKDV_OK;
}

// The ordered output's buffers for at most max_segs segments, max_runs runs of
// ranks and np points.
hipError_t ensure_output(tkdv_ctx *ctx, unsigned long long max_segs, unsigned long long max_runs, int np)
{
    hipError_t e = ensure(ctx->seg, cuts_bytes(np));
    if (e == hipSuccess) e = ensure(ctx->runs, cuts_bytes(np));
    if (e == hipSuccess) e = ensure(ctx->seg_cnt, sizeof(unsigned int) * max_segs);
    if (e == hipSuccess) e = ensure(ctx->seg_base, sizeof(unsigned long long) * (max_segs + 1));
    if (e == hipSuccess) e = ensure(ctx->ranks, sizeof(PointRanks) * (size_t)np);
    if (e == hipSuccess) e = ensure(ctx->run_stats, sizeof(RunStats) * max_runs);
    return e;
}

// One sampling call with the context's buffers, grown as the call needs.
tkdv_status run(tkdv_ctx *ctx, Call &call, int precision, int proposal, float *d_xhat,
                unsigned long long *d_index, hipStream_t st, std::vector<PointResult> *res_out,
                std::vector<DevCounters> *cnt_out, unsigned long long *n_deferred_out,
                float *dbg_xhat, float *dbg_t, float *dbg_s3, float *dbg_la, float *dbg_lu,
                bool stats)
{
    const int np = (int)call.pts.size();
    const unsigned long long defer_cap =
        std::min<unsigned long long>(1ull << 26, std::max<unsigned long long>(1ull << 20, call.total_tiles));
    HIP_TRY(ctx, ensure(ctx->bitmap, call.bitmap_words * 4));
    HIP_TRY(ctx, ensure(ctx->defer_list, defer_cap * 8));
    const CallState cs(np);
    const PointList pl(np, call.plist.size());
    HIP_TRY(ctx, ensure(ctx->state, cs.bytes));
    HIP_TRY(ctx, ensure(ctx->points, pl.bytes));
    HIP_TRY(ctx, ensure_output(ctx, call.max_segs, call.max_runs, np));
    HIP_TRY(ctx, ensure_host(ctx->h_points, ctx->h_points_bytes, pl.bytes));
    HIP_TRY(ctx, ensure_host(ctx->h_state, ctx->h_state_bytes, cs.back()));
    for (int ki = 0; ki < kNumK; ++ki) {
        if (call.plist_n[ki] == 0) continue;
        tkdv_status s = build_tables(ctx, 8 << ki);
        if (s != TKDV_OK) return s;
    }
    Workspace w;
    w.bitmap = reinterpret_cast<uint32_t *>(ctx->bitmap.p);
    w.defer_list = reinterpret_cast<unsigned long long *>(ctx->defer_list.p);
    w.defer_cap = defer_cap;
    w.state = static_cast<char *>(ctx->state.p);
    w.points = static_cast<char *>(ctx->points.p);
    w.seg = reinterpret_cast<Cuts *>(ctx->seg.p);
    w.runs = reinterpret_cast<Cuts *>(ctx->runs.p);
    w.ranks = reinterpret_cast<PointRanks *>(ctx->ranks.p);
    w.seg_cnt = reinterpret_cast<unsigned int *>(ctx->seg_cnt.p);
    w.seg_base = reinterpret_cast<unsigned long long *>(ctx->seg_base.p);
    w.run_stats = reinterpret_cast<RunStats *>(ctx->run_stats.p);
    if (res_out) res_out->resize(np);
    if (cnt_out) cnt_out->resize(np);
    return launch_sequence(ctx, view_of(call), w, precision, proposal, d_xhat, d_index, st,
                           res_out ? res_out->data() : nullptr, cnt_out ? cnt_out->data() : nullptr,
                           n_deferred_out, dbg_xhat, dbg_t, dbg_s3, dbg_la, dbg_lu, stats);
}

float key_to_float(unsigned int k)
{
    uint32_t u = (k & 0x80000000u) ? (k & 0x7FFFFFFFu) : ~k;
    float f;
    std::memcpy(&f, &u, 4);
    return f;
}

// The extremes against 4 sigma: the peak from its u~ key, u = sqrt(2 E0/pi) u~.
void fill_extremes(tkdv_stats &s, const DevPoint &P, const PointResult &r)
{
    s.n_exceed_4sigma = r.n_exceed4;
    s.n_samples_4sigma = r.n_max4;
    if (r.peak_key) {
        s.peak_u = std::sqrt(2.0 * P.E0 / kPi) * (double)key_to_float(r.peak_key);
        s.peak_index = r.peak_index;
    } else {
        s.peak_u = -INFINITY;
        s.peak_index = UINT64_MAX;
    }
}

void fill_stats(tkdv_stats &s, const DevPoint &P, const PointResult &r, const DevCounters &c, int mode)
{
    std::memset(&s, 0, sizeof(s));
    const int K = P.K, N = 4 * K;
    if (mode == TKDV_COUNT_ACCEPTED && P.target != ~0ull && r.n_accepted >= P.target && P.target > 0)
        s.n_proposed = c.last_index - P.i0 + 1;
    else
        s.n_proposed = r.n_processed;
    s.n_accepted = r.n_samples;
    s.n_written = r.n_written;
    const CounterShard ct = shard_totals(c);
    s.n_fp64_fixups = ct.deferred;
    s.n_M_violations = ct.violations;
    s.n_exceed_2sigma = r.n_exceed;
    s.n_grid_values = r.n_samples * (uint64_t)N;
    s.max_log_a = ct.max_log_a_key ? (double)key_to_float(ct.max_log_a_key) : -INFINITY;
    s.S1 = r.S1;
    s.S2 = r.S2;
    s.S3 = r.S3;
    s.S4 = r.S4;
    if (s.n_grid_values > 0) {
        const double n = (double)s.n_grid_values;
        const double m2 = r.S2 / n, m3 = r.S3 / n, m4 = r.S4 / n;
        s.skewness = m3 / std::pow(m2, 1.5);
        s.kurtosis = m4 / (m2 * m2);
        s.p_exceed_2sigma = (double)r.n_exceed / n;
    }
    const double umax = std::sqrt(2.0 * K * P.E0 / kPi);
    s.hist_lo = -umax;
    s.hist_hi = umax;
    for (int b = 0; b < TKDV_NBINS; ++b) s.hist_u0[b] = r.hist[b];
    s.log_M_used = P.log_M64;
    fill_extremes(s, P, r);
}

tkdv_status prepare(tkdv_ctx *ctx, Call &call, int n_points, const tkdv_point *pts, int proposal,
                    const tkdv_plan *plans, const uint64_t *n, int mode, uint64_t max_proposals,
                    int precision, const uint64_t *capacity, const uint64_t *out_offset, uint64_t row_stride,
                    uint64_t i0)
{
    if (n_points < 1) return set_err(ctx, TKDV_E_ARG, "n_points must be >= 1");
    if (proposal != TKDV_PROP_UNIFORM && proposal != TKDV_PROP_SIGMA && proposal != TKDV_PROP_MIXTURE)
        return set_err(ctx, TKDV_E_ARG, "bad proposal");
    if (proposal == TKDV_PROP_MIXTURE && !plans) return set_err(ctx, TKDV_E_ARG, "the mixture needs its plan");
    if (precision < TKDV_FP32 || precision > TKDV_BF16X3) return set_err(ctx, TKDV_E_ARG, "bad precision");
    if (precision == TKDV_BF16) return set_err(ctx, TKDV_E_UNSUPPORTED, kBf16Refused);
    if (mode != TKDV_COUNT_PROPOSALS && mode != TKDV_COUNT_ACCEPTED) return set_err(ctx, TKDV_E_ARG, "bad mode");
    if (mode == TKDV_COUNT_ACCEPTED && max_proposals == 0)
        return set_err(ctx, TKDV_E_ARG, "accepted-count mode needs max_proposals > 0");
    call.pts.resize(n_points);
    call.plist_n.assign(kNumK, 0);
    call.plist_off.assign(kNumK, 0);
    std::vector<std::vector<int>> by_k(kNumK);
    unsigned long long bm = 0, tiles = 0, runs = 0;
    for (int p = 0; p < n_points; ++p) {
        tkdv_status s = check_point(ctx, pts[p]);
        if (s != TKDV_OK) return s;
        tkdv_plan pl;
        if (plans) {
            pl = plans[p];
            if (pl.proposal != proposal) return set_err(ctx, TKDV_E_ARG, "plan was made for another proposal");
            if (!std::isfinite(pl.log_M) || !(pl.alpha_star > 0.0))
                return set_err(ctx, TKDV_E_ARG, "plan has non-finite log_M or alpha*");
        } else {
            s = (tkdv_status)plan_point_host(&pts[p], proposal, 2, &pl);
            if (s != TKDV_OK) return set_err(ctx, s, "planning failed");
        }
        DevPoint &d = call.pts[p];
        fill_devpoint(d, pts[p], pl, proposal, precision);
        const uint64_t ncov = mode == TKDV_COUNT_PROPOSALS ? n[p] : max_proposals;
        if (i0 + ncov < i0 || i0 + ncov >= (1ull << 40))
            return set_err(ctx, TKDV_E_ARG, "proposal indices must stay below 2^40");
        d.i0 = i0;
        d.n = ncov;
        d.n_tiles = (ncov + kTile - 1) / kTile;
        d.target = mode == TKDV_COUNT_ACCEPTED ? n[p] : ~0ull;
        d.static_tiles = static_share(d.n_tiles, mode == TKDV_COUNT_ACCEPTED
                                                     ? std::max(kAlwaysTiles / (uint64_t)n_points, n[p] / kTile)
                                                     : d.n_tiles,
                                      n_points);
        d.bm_off = bm;
        d.out_off = out_offset ? out_offset[p] : 0;
        d.capacity = capacity ? capacity[p] : 0;
        d.row_stride = row_stride;
        bm += d.n_tiles;
        runs += max_runs(d.K, std::min(d.target, d.n));
        tiles += d.n_tiles;
        by_k[kindex(pts[p].K)].push_back(p);
    }
    call.plist.clear();
    for (int ki = 0; ki < kNumK; ++ki) {
        call.plist_off[ki] = (int)call.plist.size();
        call.plist_n[ki] = (int)by_k[ki].size();
        call.plist.insert(call.plist.end(), by_k[ki].begin(), by_k[ki].end());
    }
    call.bitmap_words = bm;
    call.max_segs = max_segments(bm, n_points);
    call.max_runs = runs;
    call.total_tiles = tiles;
    return TKDV_OK;
}

// Learned proposal: host FP64 set-up of the point's constants and tables,
// uploaded to the context, and the point's decision window widened by the
// error bound of the FP32 log q_mix.
tkdv_status prepare_mixture(tkdv_ctx *ctx, Call &call, const tkdv_point &pt, const tkdv_plan &plan,
                            const tkdv_mixture *mix, int precision, hipStream_t st)
{
    if (!mix) return set_err(ctx, TKDV_E_ARG, "mixture is NULL");
    if (pt.K > 32) return set_err(ctx, TKDV_E_UNSUPPORTED, "the mixture sampler supports K in {8,16,32}");
    if (plan.proposal != TKDV_PROP_MIXTURE) return set_err(ctx, TKDV_E_ARG, "plan was made for another proposal");
    MixHost mh;
    if (mh.init(pt, plan, *mix) != TKDV_OK) return set_err(ctx, TKDV_E_ARG, "invalid mixture parameters");
    if (!(mh.kappa() <= 1e5)) return set_err(ctx, TKDV_E_ARG, "mixture too ill-conditioned (lambda_max(G) > 1e5)");
    std::vector<DevMix> dm(1);
    std::vector<uint8_t> tab;
    mix_device_data(mh, dm[0], tab);
    dm[0].tab_off = 0;
    HIP_TRY(ctx, ensure(ctx->mix, sizeof(DevMix)));
    HIP_TRY(ctx, ensure(ctx->mix_tab, tab.size()));
    HIP_TRY(ctx, hipMemcpyAsync(ctx->mix.p, dm.data(), sizeof(DevMix), hipMemcpyHostToDevice, st));
    HIP_TRY(ctx, hipMemcpyAsync(ctx->mix_tab.p, tab.data(), tab.size(), hipMemcpyHostToDevice, st));
    HIP_TRY(ctx, hipStreamSynchronize(st));  // the host vectors go out of scope
    set_window(call.pts[0], window(pt, TKDV_PROP_MIXTURE, precision, plan.alpha_star, plan.log_M,
                                   mix_window_extra(mh, precision)));
    return TKDV_OK;
}

// Stats of a finished sweep point.
void fill_stats_sweep(tkdv_stats &s, const DevPoint &P, const SweepState &w)
{
    std::memset(&s, 0, sizeof(s));
    const int K = P.K, N = 4 * K;
    s.n_proposed = w.n_proposed;
    s.n_accepted = w.accepted;
    s.n_written = w.written;
    s.n_fp64_fixups = w.n_fixups;
    s.n_M_violations = w.n_violations;
    s.n_exceed_2sigma = w.total.n_exceed;
    s.n_grid_values = w.accepted * (uint64_t)N;
    s.max_log_a = w.max_log_a_key ? (double)key_to_float(w.max_log_a_key) : -INFINITY;
    s.S1 = w.total.S1;
    s.S2 = w.total.S2;
    s.S3 = w.total.S3;
    s.S4 = w.total.S4;
    if (s.n_grid_values > 0) {
        const double n = (double)s.n_grid_values;
        const double m2 = s.S2 / n, m3 = s.S3 / n, m4 = s.S4 / n;
        s.skewness = m3 / std::pow(m2, 1.5);
        s.kurtosis = m4 / (m2 * m2);
        s.p_exceed_2sigma = (double)w.total.n_exceed / n;
    }
    const double umax = std::sqrt(2.0 * K * P.E0 / kPi);
    s.hist_lo = -umax;
    s.hist_hi = umax;
    for (int b = 0; b < TKDV_NBINS; ++b) s.hist_u0[b] = w.total.hist[b];
    s.log_M_used = P.log_M64;
    fill_extremes(s, P, w.total);
}

int prec_index(int precision) { return precision < 0 || precision > 2 ? 0 : precision; }

// Windows captured into one graph (one launch, one host synchronisation).  Most
// sweeps take two or three; the windows after them do nothing but launch, some
// 60 us each, and are captured and instantiated all the same: with 16 of them a map
// of 64 cells took 3.8 ms, with 4 3.0, and a sweep of 24 points 12.2 and 11.0.  A
// look at the state costs some 13 us: sweeps in fixed windows of 65536 proposals
// (one point, K = 16) take 0.66 ms with 4 and 1.01 with 16 for 5 windows, 2.93 and
// 3.10 for 41, 6.75 and 6.70 for 101, 25.6 and 24.3 for 400; of 2^20 proposals 0.94
// and 1.24, 4.99 and 5.08, 11.8 and 11.9, 46.5 and 45.4.
constexpr int kSweepGraphWindows = 4;

tkdv_status sweep(tkdv_ctx *ctx, int np, const tkdv_point *pts, const tkdv_plan *plans, const uint64_t *targets,
                  const uint64_t *maxp, int precision, const tkdv_launch_cfg *cfg, float *d_xhat,
                  uint64_t *d_index, const uint64_t *capacity, const uint64_t *out_offset, tkdv_stats *h_stats,
                  hipStream_t user_st)
{
    if (np < 1) return set_err(ctx, TKDV_E_ARG, "n_points must be >= 1");
    if (!pts || !targets || !maxp || !h_stats) return set_err(ctx, TKDV_E_ARG, "NULL argument");
    if (precision < TKDV_FP32 || precision > TKDV_BF16X3) return set_err(ctx, TKDV_E_ARG, "bad precision");
    if (precision == TKDV_BF16) return set_err(ctx, TKDV_E_UNSUPPORTED, kBf16Refused);
    Call call;
    call.pts.resize(np);
    call.plist_n.assign(kNumK, 0);
    call.plist_off.assign(kNumK, 0);
    std::vector<std::vector<int>> by_k(kNumK);
    std::vector<SweepState> sw(np);
    tkdv_launch_cfg kcfg[kNumK];
    bool use_graph = true, adaptive = np <= 1024;
    for (int ki = 0; ki < kNumK; ++ki) kcfg[ki] = cfg ? *cfg : ctx->lcfg[ki][prec_index(precision)];
    unsigned long long first_words = 0, sum_maxp = 0;
    for (int p = 0; p < np; ++p) {
        tkdv_status s = check_point(ctx, pts[p]);
        if (s != TKDV_OK) return s;
        if (targets[p] < 1 || maxp[p] < 1 || maxp[p] >= (1ull << 40))
            return set_err(ctx, TKDV_E_ARG, "targets must be >= 1 and max_proposals in [1, 2^40)");
        tkdv_plan pl;
        if (plans) {
            pl = plans[p];
            if (pl.proposal != TKDV_PROP_SIGMA) return set_err(ctx, TKDV_E_ARG, "the sweep takes Sigma plans");
        } else {
            s = (tkdv_status)plan_point_host(&pts[p], TKDV_PROP_SIGMA, 2, &pl);
            if (s != TKDV_OK) return set_err(ctx, s, "planning failed");
        }
        const int ki = kindex(pts[p].K);
        const tkdv_launch_cfg &lc = kcfg[ki];
        if (lc.window < 65536 || lc.window % 65536 != 0 || lc.window > (1ull << 34) || lc.blocks_per_cu < 0 ||
            lc.variant < 0 || lc.variant >= TKDV_DECIDE_VARIANTS)
            return set_err(ctx, TKDV_E_ARG, "window must be a multiple of 65536 in [65536, 2^34], variant in range");
        use_graph = use_graph && lc.use_graph;
        adaptive = adaptive && lc.adaptive;
        DevPoint &d = call.pts[p];
        fill_devpoint(d, pts[p], pl, TKDV_PROP_SIGMA, precision);
        const uint64_t W = lc.window;
        d.i0 = 0;
        d.n = std::min<uint64_t>(W, maxp[p]);
        d.n_tiles = (d.n + kTile - 1) / kTile;
        d.target = targets[p];
        d.static_tiles = static_share(d.n_tiles, targets[p] / kTile, np);
        d.bm_off = first_words;
        d.out_off = out_offset ? out_offset[p] : 0;
        d.capacity = capacity ? capacity[p] : 0;
        d.row_stride = 2 * TKDV_KMAX;
        first_words += d.n_tiles;
        sum_maxp += maxp[p];
        std::memset(&sw[p], 0, sizeof(SweepState));
        sw[p].i_start = 0;
        sw[p].i_end = maxp[p];
        sw[p].window = W;
        sw[p].target = targets[p];
        sw[p].capacity = d.capacity;
        sw[p].out_off = d.out_off;
        by_k[ki].push_back(p);
    }
    // the window's accept bitmap: the first windows, or (adaptive) a pool of up
    // to 2^33 proposals shared by the points' later windows, plus 65536
    // proposals per point of rounding
    unsigned long long pool_words = first_words;
    if (adaptive) pool_words = std::max<unsigned long long>(first_words, std::min<unsigned long long>(
                                                                              (1ull << 33) / kTile, sum_maxp / kTile));
    const unsigned long long bm_words = pool_words + (unsigned long long)np * 2048;
    const unsigned long long max_segs = max_segments(bm_words, np);
    unsigned long long n_runs = 0;  // most of a window
    for (int p = 0; p < np; ++p) n_runs += max_runs(pts[p].K, std::min(targets[p], maxp[p]));
    call.plist.clear();
    for (int ki = 0; ki < kNumK; ++ki) {
        call.plist_off[ki] = (int)call.plist.size();
        call.plist_n[ki] = (int)by_k[ki].size();
        call.plist.insert(call.plist.end(), by_k[ki].begin(), by_k[ki].end());
    }
    hipStream_t sst = ctx->sweep_stream;
    const unsigned long long defer_cap = std::min<unsigned long long>(1ull << 26, std::max<unsigned long long>(1ull << 20, bm_words));
    HIP_TRY(ctx, ensure(ctx->bitmap, bm_words * 4));
    HIP_TRY(ctx, ensure(ctx->defer_list, defer_cap * 8));
    const CallState cs(np);
    const PointList pl(np, call.plist.size());
    char *points = nullptr, *state = nullptr;
    HIP_TRY(ctx, ensure(ctx->state, cs.bytes));
    HIP_TRY(ctx, ensure(ctx->points, pl.bytes));
    state = static_cast<char *>(ctx->state.p);
    points = static_cast<char *>(ctx->points.p);
    HIP_TRY(ctx, ensure_output(ctx, max_segs, n_runs, np));
    HIP_TRY(ctx, ensure(ctx->sweep, sizeof(SweepState) * np));
    HIP_TRY(ctx, ensure(ctx->active, sizeof(SweepGlobal)));
    for (int ki = 0; ki < kNumK; ++ki)
        if (call.plist_n[ki]) {
            tkdv_status s = build_tables(ctx, 8 << ki);
            if (s != TKDV_OK) return s;
        }
    SweepGlobal g0;
    std::memset(&g0, 0, sizeof(g0));
    g0.pool_tiles = pool_words;
    g0.active = (unsigned long long)np;
    g0.defer_cap = defer_cap;
    g0.adaptive = adaptive ? 1 : 0;
    // the caller's stream has finished its earlier work before the sweep reads
    // or writes the caller's buffers
    HIP_TRY(ctx, hipEventRecord(ctx->join[0], user_st));
    HIP_TRY(ctx, hipStreamWaitEvent(sst, ctx->join[0], 0));
    HIP_TRY(ctx, hipMemcpyAsync(points, call.pts.data(), sizeof(DevPoint) * np, hipMemcpyHostToDevice, sst));
    HIP_TRY(ctx, hipMemcpyAsync(points + pl.plist, call.plist.data(), sizeof(int) * call.plist.size(),
                                hipMemcpyHostToDevice, sst));
    HIP_TRY(ctx, hipMemcpyAsync(ctx->sweep.p, sw.data(), sizeof(SweepState) * np, hipMemcpyHostToDevice, sst));
    HIP_TRY(ctx, hipMemcpyAsync(ctx->active.p, &g0, sizeof(g0), hipMemcpyHostToDevice, sst));
    HIP_TRY(ctx, hipStreamSynchronize(sst));  // host vectors are pageable and go out of scope

    SweepGlobal *dG = reinterpret_cast<SweepGlobal *>(ctx->active.p);
    KernelArgs a;
    std::memset(&a, 0, sizeof(a));
    set_state(a, state, cs);
    a.pts = reinterpret_cast<const DevPoint *>(points);
    a.n_points = np;
    a.bitmap = reinterpret_cast<uint32_t *>(ctx->bitmap.p);
    a.defer_list = reinterpret_cast<unsigned long long *>(ctx->defer_list.p);
    a.defer_cap = defer_cap;
    a.d_active = &dG->active;
    a.seg = reinterpret_cast<Cuts *>(ctx->seg.p);
    a.runs = reinterpret_cast<Cuts *>(ctx->runs.p);
    a.ranks = reinterpret_cast<PointRanks *>(ctx->ranks.p);
    a.seg_cnt = reinterpret_cast<unsigned int *>(ctx->seg_cnt.p);
    a.seg_base = reinterpret_cast<unsigned long long *>(ctx->seg_base.p);
    a.run_stats = reinterpret_cast<RunStats *>(ctx->run_stats.p);
    const int *d_plist = reinterpret_cast<const int *>(points + pl.plist);
    // one window: every launch is sized for the largest window (persistent
    // kernels), the device holds the current window's extent
    auto window = [&]() -> tkdv_status {
        HIP_TRY(ctx, launch_fill_u32(state, cs.bytes / 4, 0u, sst));
        for (int ki = 0; ki < kNumK; ++ki) {
            if (call.plist_n[ki] == 0) continue;
            const int K = 8 << ki;
            a.blocks_per_cu = kcfg[ki].blocks_per_cu;
            // the tile variants other than 0 run with BF16x3 products only
            decide_tables(ctx, ki, precision, precision == TKDV_BF16X3 ? kcfg[ki].variant : 0, a.phi_hi,
                          a.phi_lo);
            HIP_TRY(ctx, launch_decide_variant(K, precision, TKDV_PROP_SIGMA, kcfg[ki].variant, a,
                                               d_plist + call.plist_off[ki], call.plist_n[ki], ctx->n_cu,
                                               pool_words, sst, nullptr));
        }
        bool plan = true;  // the first launch lays out the segments
        for (int ki = 0; ki < kNumK; ++ki) {
            if (call.plist_n[ki] == 0) continue;
            HIP_TRY(ctx, launch_fixup(8 << ki, a, plan, ctx->n_cu, sst));
            plan = false;
        }
        HIP_TRY(ctx, launch_segments(a, max_segs, ctx->n_cu, sst));
        for (int ki = 0; ki < kNumK; ++ki) {
            if (call.plist_n[ki] == 0) continue;
            a.phi_hi = ki >= 3 ? ctx->qstat[ki - 3].p : ctx->phi_f32[ki].p;
            HIP_TRY(ctx, launch_materialize(8 << ki, TKDV_PROP_SIGMA, a, n_runs, d_xhat,
                                            reinterpret_cast<unsigned long long *>(d_index), ctx->n_cu, sst));
        }
        HIP_TRY(ctx, launch_finalize(a, sst));
        HIP_TRY(ctx, launch_window_advance(reinterpret_cast<DevPoint *>(points), a.cnt, a.res,
                                           reinterpret_cast<SweepState *>(ctx->sweep.p), np, dG, a.defer_count, sst));
        return TKDV_OK;
    };
    // kSweepGraphWindows windows per launch (a window with no point left does
    // nothing); the host looks at the device state once per launch
    auto batch = [&]() -> tkdv_status {
        for (int w = 0; w < kSweepGraphWindows; ++w) {
            tkdv_status s = window();
            if (s != TKDV_OK) return s;
        }
        return TKDV_OK;
    };
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    auto release = [&]() {
        if (exec) (void)hipGraphExecDestroy(exec);
        if (graph) (void)hipGraphDestroy(graph);
        exec = nullptr;
        graph = nullptr;
    };
    if (use_graph) {
        HIP_TRY(ctx, hipStreamBeginCapture(sst, hipStreamCaptureModeThreadLocal));
        tkdv_status s = batch();
        hipError_t e = hipStreamEndCapture(sst, &graph);
        if (s != TKDV_OK) {
            release();
            return s;
        }
        if (e != hipSuccess) {
            release();
            return set_err(ctx, TKDV_E_DEVICE, std::string("graph capture: ") + hipGetErrorString(e));
        }
        e = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
        if (e != hipSuccess) {
            release();
            return set_err(ctx, TKDV_E_DEVICE, std::string("graph instantiate: ") + hipGetErrorString(e));
        }
    }
    std::memset(&ctx->timing, 0, sizeof(ctx->timing));
    for (int ki = 0; ki < kNumK; ++ki)  // the largest K of the sweep sets the reported workgroup size
        if (!by_k[ki].empty()) ctx->timing.decide_block = decide_variant_block(8 << ki, kcfg[ki].variant);
    SweepGlobal *poll = reinterpret_cast<SweepGlobal *>(ctx->h_poll);
    tkdv_status st_out = TKDV_OK;
    int launches = 0;
    // a point takes at least one window per 2^34 proposals of its range
    const unsigned long long max_launches = 1 + (sum_maxp / 65536 + (unsigned long long)np) / kSweepGraphWindows;
    hipError_t e = hipEventRecord(ctx->ev[0], sst);
    for (unsigned long long L = 0; L < max_launches && e == hipSuccess && st_out == TKDV_OK; ++L) {
        if (use_graph) e = hipGraphLaunch(exec, sst);
        else st_out = batch();
        if (e != hipSuccess || st_out != TKDV_OK) break;
        ++launches;
        if ((e = hipMemcpyAsync(poll, dG, sizeof(SweepGlobal), hipMemcpyDeviceToHost, sst)) != hipSuccess) break;
        if ((e = hipStreamSynchronize(sst)) != hipSuccess) break;
        if (poll->overflow) {
            st_out = set_err(ctx, TKDV_E_CAPACITY, "FP64 re-decision list overflowed in a sweep window");
            break;
        }
        if (poll->active == 0) break;
    }
    if (e == hipSuccess) e = hipEventRecord(ctx->ev[1], sst);
    if (e == hipSuccess) e = hipEventSynchronize(ctx->ev[1]);
    release();
    if (e != hipSuccess) return set_err(ctx, TKDV_E_DEVICE, std::string("sweep: ") + hipGetErrorString(e));
    if (st_out != TKDV_OK) return st_out;
    float ms = 0.0f;
    HIP_TRY(ctx, hipEventElapsedTime(&ms, ctx->ev[0], ctx->ev[1]));
    ctx->timing.total_ms = ms;
    ctx->timing.windows = (int)poll->windows;
    ctx->timing.graph_launches = launches;
    int nk = 0;
    for (int ki = 0; ki < kNumK; ++ki) nk += call.plist_n[ki] ? 1 : 0;
    ctx->timing.decide_launches = (int)poll->windows * nk;
    HIP_TRY(ctx, hipMemcpy(sw.data(), ctx->sweep.p, sizeof(SweepState) * np, hipMemcpyDeviceToHost));
    for (int p = 0; p < np; ++p) fill_stats_sweep(h_stats[p], call.pts[p], sw[p]);
    // later work on the caller's stream sees the sweep's outputs
    HIP_TRY(ctx, hipEventRecord(ctx->join[1], sst));
    HIP_TRY(ctx, hipStreamWaitEvent(user_st, ctx->join[1], 0));
    return TKDV_OK;
}

}  // namespace

namespace tkdv {
int ctx_device(const tkdv_ctx *ctx) { return ctx->device; }
tkdv_status record_error(tkdv_status st, const std::string &msg) { return set_err(nullptr, st, msg); }
}  // namespace tkdv

extern "C" {

tkdv_status tkdv_create(int hip_device, tkdv_ctx **out)
{
    if (!out) return set_err(nullptr, TKDV_E_ARG, "out is NULL");
    *out = nullptr;
    int n = 0;
    hipError_t e = hipGetDeviceCount(&n);
    if (e != hipSuccess || n < 1) return set_err(nullptr, TKDV_E_DEVICE, "no HIP device");
    if (hip_device < 0 || hip_device >= n) return set_err(nullptr, TKDV_E_ARG, "bad device index");
    e = hipSetDevice(hip_device);
    if (e != hipSuccess) return set_err(nullptr, TKDV_E_DEVICE, hipGetErrorString(e));
    hipDeviceProp_t prop;
    e = hipGetDeviceProperties(&prop, hip_device);
    if (e != hipSuccess) return set_err(nullptr, TKDV_E_DEVICE, hipGetErrorString(e));
    tkdv_ctx *ctx = new tkdv_ctx();
    ctx->device = hip_device;
    ctx->n_cu = prop.multiProcessorCount;
    ctx->arch = prop.gcnArchName;
    for (auto &row : ctx->lcfg)
        for (auto &c : row) c = tkdv_launch_cfg{0, 1, 1ull << 26, 0, 1};
    e = hipStreamCreateWithFlags(&ctx->sweep_stream, hipStreamNonBlocking);
    if (e == hipSuccess) e = hipEventCreateWithFlags(&ctx->join[0], hipEventDisableTiming);
    if (e == hipSuccess) e = hipEventCreateWithFlags(&ctx->join[1], hipEventDisableTiming);
    if (e == hipSuccess) e = hipHostMalloc(&ctx->h_poll, 256, hipHostMallocDefault);
    if (e != hipSuccess) {
        tkdv_destroy(ctx);
        return set_err(nullptr, TKDV_E_DEVICE, hipGetErrorString(e));
    }
    for (hipEvent_t &ev : ctx->ev) {
        e = hipEventCreate(&ev);
        if (e != hipSuccess) {
            tkdv_destroy(ctx);
            return set_err(nullptr, TKDV_E_DEVICE, hipGetErrorString(e));
        }
    }
    // set-up of tkdv_sample_noalloc: the device address of this GPU's fixed
    // scratch array, every K's synthesis tables and the one-point pinned
    // staging, so that its calls find everything in place
    e = scratch_init(hip_device);
    if (e == hipSuccess) e = ensure_host(ctx->h_points, ctx->h_points_bytes, PointList(1, 1).bytes);
    if (e == hipSuccess) e = ensure_host(ctx->h_state, ctx->h_state_bytes, CallState(1).back());
    if (e != hipSuccess) {
        tkdv_destroy(ctx);
        return set_err(nullptr, TKDV_E_DEVICE, std::string("set-up of the fixed scratch: ") + hipGetErrorString(e));
    }
    for (int ki = 0; ki < kNumK; ++ki) {
        const tkdv_status st = build_tables(ctx, 8 << ki);
        if (st != TKDV_OK) {
            const std::string msg = ctx->last_error;
            tkdv_destroy(ctx);
            return set_err(nullptr, st, msg);
        }
    }
    *out = ctx;
    return TKDV_OK;
}

tkdv_status tkdv_sample_noalloc(tkdv_ctx *ctx, const tkdv_point *pt, tkdv_proposal proposal, const tkdv_plan *plan,
                                uint64_t n, tkdv_count_mode mode, uint64_t max_proposals, tkdv_precision precision,
                                float *d_xhat, uint64_t *d_index, uint64_t capacity, tkdv_stats *h_stats,
                                void *stream)
{
    if (!ctx) return set_err(nullptr, TKDV_E_ARG, "ctx is NULL");
    if (!pt || !plan || !h_stats) return set_err(ctx, TKDV_E_ARG, "NULL argument (the plan is required)");
    tkdv_status s = check_point(ctx, *pt);
    if (s != TKDV_OK) return s;
    if (proposal != TKDV_PROP_UNIFORM && proposal != TKDV_PROP_SIGMA)
        return set_err(ctx, TKDV_E_ARG, "proposal must be UNIFORM or SIGMA");
    if (plan->proposal != proposal) return set_err(ctx, TKDV_E_ARG, "plan was made for another proposal");
    if (!std::isfinite(plan->log_M) || !(plan->alpha_star > 0.0))
        return set_err(ctx, TKDV_E_ARG, "plan has non-finite log_M or alpha*");
    if (precision != TKDV_FP32 && precision != TKDV_BF16X3)
        return set_err(ctx, precision == TKDV_BF16 ? TKDV_E_UNSUPPORTED : TKDV_E_ARG, kBf16Refused);
    if (mode != TKDV_COUNT_PROPOSALS && mode != TKDV_COUNT_ACCEPTED) return set_err(ctx, TKDV_E_ARG, "bad mode");
    if (mode == TKDV_COUNT_ACCEPTED && max_proposals == 0)
        return set_err(ctx, TKDV_E_ARG, "accepted-count mode needs max_proposals > 0");
    const uint64_t covered = mode == TKDV_COUNT_PROPOSALS ? n : max_proposals;
    if (covered > kScratchMaxProposals)
        return set_err(ctx, TKDV_E_ARG,
                       "tkdv_sample_noalloc covers at most 2^26 proposals per call (its fixed scratch); "
                       "use tkdv_sample for more");
    HIP_TRY(ctx, hipSetDevice(ctx->device));
    const int ki = kindex(pt->K);
    char *base = static_cast<char *>(scratch_ptr(ctx->device));
    const CallState cs(1);
    const PointList list(1, 1);
    if (!base || !ctx->phi_hi[ki].p || !ctx->h_points || ctx->h_points_bytes < list.bytes ||
        ctx->h_state_bytes < cs.back())
        return set_err(ctx, TKDV_E_DEVICE, "the context's set-up of the fixed scratch is missing");
    if (n == 0) {
        std::memset(h_stats, 0, sizeof(*h_stats));
        const double umax = std::sqrt(2.0 * pt->K * pt->E0 / kPi);
        h_stats->hist_lo = -umax;
        h_stats->hist_hi = umax;
        h_stats->max_log_a = -INFINITY;
        h_stats->log_M_used = plan->log_M;
        return TKDV_OK;
    }
    // the scratch: accept bitmap, FP64 re-decision list, then the small
    // records, each 256-byte aligned
    const uint64_t n_tiles = (covered + kTile - 1) / kTile;
    auto carve = [&](size_t &off, size_t bytes) {
        char *p = base + off;
        off += (bytes + 255) & ~(size_t)255;
        return p;
    };
    size_t off = 0;
    Workspace w;
    w.bitmap = reinterpret_cast<uint32_t *>(carve(off, (kScratchMaxProposals / 32) * 4));
    w.defer_list = reinterpret_cast<unsigned long long *>(carve(off, kScratchDeferCap * 8));
    w.defer_cap = kScratchDeferCap;
    w.state = carve(off, cs.bytes);
    w.points = carve(off, list.bytes);
    const size_t max_segs = max_segments(kScratchMaxProposals / 32, 1);
    w.seg = reinterpret_cast<Cuts *>(carve(off, cuts_bytes(1)));
    w.runs = reinterpret_cast<Cuts *>(carve(off, cuts_bytes(1)));
    w.seg_cnt = reinterpret_cast<unsigned int *>(carve(off, max_segs * sizeof(unsigned int)));
    w.seg_base = reinterpret_cast<unsigned long long *>(carve(off, (max_segs + 1) * 8));
    w.ranks = reinterpret_cast<PointRanks *>(carve(off, sizeof(PointRanks)));
    w.run_stats = reinterpret_cast<RunStats *>(carve(off, max_runs(pt->K, kScratchMaxProposals) * sizeof(RunStats)));
    if (off > kScratchBytes) return set_err(ctx, TKDV_E_CAPACITY, "fixed scratch layout exceeds its size");
    tkdv_plan pl = *plan;
    const int plist0 = 0;
    for (int raise = 0;; ++raise) {
        DevPoint d;
        fill_devpoint(d, *pt, pl, proposal, precision);
        d.i0 = 0;
        d.n = covered;
        d.n_tiles = n_tiles;
        d.target = mode == TKDV_COUNT_ACCEPTED ? n : ~0ull;
        d.static_tiles =
            static_share(n_tiles, mode == TKDV_COUNT_ACCEPTED ? std::max(kAlwaysTiles, n / kTile) : n_tiles, 1);
        d.bm_off = 0;
        d.out_off = 0;
        d.capacity = capacity;
        d.row_stride = 2 * (uint64_t)pt->K;
        CallView v;
        v.pts = &d;
        v.np = 1;
        v.plist = &plist0;
        v.plist_len = 1;
        for (int q = 0; q < kNumK; ++q) v.plist_off[q] = v.plist_n[q] = 0;
        v.plist_n[ki] = 1;
        v.max_segs = max_segments(n_tiles, 1);
        v.max_runs = max_runs(pt->K, std::min(d.target, d.n));
        PointResult res;
        DevCounters cnt;
        s = launch_sequence(ctx, v, w, precision, proposal, d_xhat, reinterpret_cast<unsigned long long *>(d_index),
                            (hipStream_t)stream, &res, &cnt, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr,
                            true);
        if (s != TKDV_OK) return s;
        fill_stats(*h_stats, d, res, cnt, mode);
        h_stats->M_raises = raise;
        if (h_stats->n_M_violations == 0 || ctx->mv_policy == TKDV_MV_COUNT) return TKDV_OK;
        if (ctx->mv_policy == TKDV_MV_FAIL || raise == kMaxRaises) return violation_error(ctx, 0, *h_stats);
        pl.log_M = raised_log_M(pl.log_M, h_stats->max_log_a, d.tau);
    }
}

tkdv_status tkdv_destroy(tkdv_ctx *ctx)
{
    if (!ctx) return TKDV_OK;
    (void)hipSetDevice(ctx->device);
    DevBuf *bufs[] = {&ctx->bitmap, &ctx->defer_list, &ctx->state, &ctx->points,
                      &ctx->seg, &ctx->seg_cnt, &ctx->seg_base, &ctx->ranks, &ctx->runs, &ctx->run_stats,
                      &ctx->mix, &ctx->mix_tab, &ctx->sweep, &ctx->active, &ctx->plan_pts, &ctx->plan_val,
                      &ctx->plan_x, &ctx->plan_ev, &ctx->plan_mix, &ctx->plan_user, &ctx->ext_keys, &ctx->ext_jmax, &ctx->ext_misc,
                      &ctx->sir_pt, &ctx->sir_w, &ctx->sir_tile, &ctx->sir_chunk, &ctx->sir_part};
    for (DevBuf *b : bufs)
        if (b->p) (void)hipFree(b->p);
    for (DevBuf *b : {&ctx->qstat[0], &ctx->qstat[1]})
        if (b->p) (void)hipFree(b->p);
    for (DevBuf *b : {&ctx->q64_hi, &ctx->q64_lo, &ctx->q64_f32})
        if (b->p) (void)hipFree(b->p);
    for (int i = 0; i < kNumK; ++i) {
        if (ctx->phi_hi[i].p) (void)hipFree(ctx->phi_hi[i].p);
        if (ctx->phi_lo[i].p) (void)hipFree(ctx->phi_lo[i].p);
        if (ctx->phi_f32[i].p) (void)hipFree(ctx->phi_f32[i].p);
        if (ctx->phi3_hi[i].p) (void)hipFree(ctx->phi3_hi[i].p);
        if (ctx->phi3_lo[i].p) (void)hipFree(ctx->phi3_lo[i].p);
        if (ctx->phi3_f32[i].p) (void)hipFree(ctx->phi3_f32[i].p);
    }
    if (ctx->h_state) (void)hipHostFree(ctx->h_state);
    if (ctx->h_points) (void)hipHostFree(ctx->h_points);
    if (ctx->h_misc) (void)hipHostFree(ctx->h_misc);
    for (hipEvent_t ev : ctx->ev)
        if (ev) (void)hipEventDestroy(ev);
    for (hipEvent_t ev : ctx->join)
        if (ev) (void)hipEventDestroy(ev);
    if (ctx->sweep_stream) (void)hipStreamDestroy(ctx->sweep_stream);
    if (ctx->h_poll) (void)hipHostFree(ctx->h_poll);
    delete ctx;
    return TKDV_OK;
}

tkdv_status tkdv_plan_point(const tkdv_point *pt, tkdv_proposal proposal, tkdv_plan *out)
{
    if (!pt || !out) return set_err(nullptr, TKDV_E_ARG, "NULL argument");
    tkdv_status s = (tkdv_status)plan_point_host(pt, proposal, 2, out);
    if (s != TKDV_OK) return set_err(nullptr, s, "planning failed");
    return TKDV_OK;
}

namespace {

// The multi-start search of k_plan_search for the points pp (mixtures and
// caller starts optional): values, final iterates [item][kPlanStride] and evaluation
// counts per item, item = point * (n_starts + n_user) + start.
tkdv_status run_plan_search(tkdv_ctx *ctx, const std::vector<PlanPoint> &pp, const std::vector<PlanMix> *mix,
                            const std::vector<double> *user, int n_user, int n_starts, uint64_t seed,
                            hipStream_t st, std::vector<double> &val, std::vector<double> &xb,
                            std::vector<int> &ev)
{
    HIP_TRY(ctx, hipSetDevice(ctx->device));
    const int per = n_starts + n_user;
    const int n_items = (int)pp.size() * per;
    HIP_TRY(ctx, ensure(ctx->plan_pts, pp.size() * sizeof(PlanPoint)));
    HIP_TRY(ctx, ensure(ctx->plan_val, (size_t)n_items * sizeof(double)));
    HIP_TRY(ctx, ensure(ctx->plan_x, (size_t)n_items * kPlanStride * sizeof(double)));
    HIP_TRY(ctx, ensure(ctx->plan_ev, (size_t)n_items * sizeof(int)));
    HIP_TRY(ctx, hipMemcpyAsync(ctx->plan_pts.p, pp.data(), pp.size() * sizeof(PlanPoint), hipMemcpyHostToDevice, st));
    PlanArgs a{};
    if (mix) {
        HIP_TRY(ctx, ensure(ctx->plan_mix, mix->size() * sizeof(PlanMix)));
        HIP_TRY(ctx, hipMemcpyAsync(ctx->plan_mix.p, mix->data(), mix->size() * sizeof(PlanMix),
                                    hipMemcpyHostToDevice, st));
        a.mix = (const PlanMix *)ctx->plan_mix.p;
    }
    if (n_user > 0) {
        HIP_TRY(ctx, ensure(ctx->plan_user, user->size() * sizeof(double)));
        HIP_TRY(ctx, hipMemcpyAsync(ctx->plan_user.p, user->data(), user->size() * sizeof(double),
                                    hipMemcpyHostToDevice, st));
        a.x_user = (const double *)ctx->plan_user.p;
    }
    a.pts = (const PlanPoint *)ctx->plan_pts.p;
    a.n_user = n_user;
    a.n_items = n_items;
    a.n_starts = n_starts;
    a.seed_lo = (uint32_t)seed;
    a.seed_hi = (uint32_t)(seed >> 32);
    a.val = (double *)ctx->plan_val.p;
    a.xbest = (double *)ctx->plan_x.p;
    a.evals = (int *)ctx->plan_ev.p;
    int max_K = 0;
    for (const PlanPoint &q : pp) max_K = std::max(max_K, q.K);
    HIP_TRY(ctx, launch_plan_search(a, max_K, st));
    val.assign(n_items, 0.0);
    xb.assign((size_t)n_items * kPlanStride, 0.0);
    ev.assign(n_items, 0);
    HIP_TRY(ctx, hipMemcpyAsync(val.data(), a.val, val.size() * sizeof(double), hipMemcpyDeviceToHost, st));
    HIP_TRY(ctx, hipMemcpyAsync(xb.data(), a.xbest, xb.size() * sizeof(double), hipMemcpyDeviceToHost, st));
    HIP_TRY(ctx, hipMemcpyAsync(ev.data(), a.evals, ev.size() * sizeof(int), hipMemcpyDeviceToHost, st));
    HIP_TRY(ctx, hipStreamSynchronize(st));
    return TKDV_OK;
}

// The best item of point w: index into val (-1 if no finite value), total evaluations.
int best_item(const std::vector<double> &val, const std::vector<int> &ev, int w, int per, long *total)
{
    int best = -1;
    *total = 0;
    for (int s = 0; s < per; ++s) {
        const int it = w * per + s;
        *total += ev[it];
        if (!std::isfinite(val[it])) continue;
        if (best < 0 || val[it] > val[best]) best = it;
    }
    return best;
}

}  // namespace

tkdv_status tkdv_plan_batch(tkdv_ctx *ctx, int32_t n_points, const tkdv_point *pts, tkdv_proposal proposal,
                            int32_t n_starts, uint64_t seed, int32_t flags, tkdv_plan *out, double *xhat_best,
                            void *stream)
{
    if (!ctx) return set_err(nullptr, TKDV_E_ARG, "ctx is NULL");
    if (n_points < 0) return set_err(ctx, TKDV_E_ARG, "n_points < 0");
    if (n_points == 0) return TKDV_OK;
    if (!pts || !out) return set_err(ctx, TKDV_E_ARG, "NULL argument");
    if (n_starts < 1 || n_starts > 256) return set_err(ctx, TKDV_E_ARG, "n_starts must be in [1, 256]");
    if (proposal != TKDV_PROP_UNIFORM && proposal != TKDV_PROP_SIGMA)
        return set_err(ctx, TKDV_E_ARG, "proposal must be UNIFORM or SIGMA");
    if (flags & ~TKDV_PLAN_SEARCH_ALWAYS) return set_err(ctx, TKDV_E_ARG, "unknown flags");
    if ((int64_t)n_points * n_starts > (int64_t)(1 << 30)) return set_err(ctx, TKDV_E_ARG, "too many starts");
    std::vector<PlanPoint> pp;
    std::vector<int> which;
    for (int p = 0; p < n_points; ++p) {
        const int st = plan_base_host(&pts[p], proposal, &out[p]);
        if (st != TKDV_OK)
            return set_err(ctx, (tkdv_status)st, "point " + std::to_string(p) + ": planning failed");
        if (xhat_best) std::fill(xhat_best + (size_t)p * 2 * TKDV_KMAX, xhat_best + (size_t)(p + 1) * 2 * TKDV_KMAX, 0.0);
        if (out[p].M_source == 0 && !(flags & TKDV_PLAN_SEARCH_ALWAYS)) continue;
        const tkdv_point &q = pts[p];
        const int K = q.K;
        PlanPoint P{};
        P.K = K;
        P.N = 4 * K;
        P.sigma = proposal == TKDV_PROP_SIGMA ? 1 : 0;
        P.point_id = q.point_id;
        P.dt0 = -q.beta_p / ((double)K * K);
        P.cH = q.beta_p * q.c32 / (q.E0 * (double)K * K);
        const double amp = std::sqrt(2.0 * q.E0 / kPi);
        P.amp3 = amp * amp * amp;
        P.a = out[p].alpha_star * q.beta_p / ((double)K * K * K);
        pp.push_back(P);
        which.push_back(p);
    }
    if (which.empty()) return TKDV_OK;
    std::vector<double> val, xb;
    std::vector<int> ev;
    tkdv_status rs = run_plan_search(ctx, pp, nullptr, nullptr, 0, n_starts, seed, (hipStream_t)stream, val, xb, ev);
    if (rs != TKDV_OK) return rs;
    for (size_t w = 0; w < which.size(); ++w) {
        const int p = which[w];
        long total = 0;
        const int bi = best_item(val, ev, (int)w, n_starts, &total);
        if (bi < 0) return set_err(ctx, TKDV_E_DEVICE, "point " + std::to_string(p) + ": search gave no value");
        out[p].log_M = val[bi];
        out[p].M_source = 2;
        out[p].n_optimiser_evals = (int32_t)std::min<long>(total, INT32_MAX);
        if (xhat_best)
            for (int m = 0; m < 2 * pts[p].K; ++m) xhat_best[(size_t)p * 2 * TKDV_KMAX + m] = xb[(size_t)bi * kPlanStride + m];
    }
    return TKDV_OK;
}

tkdv_status tkdv_plan_mixture_batch(tkdv_ctx *ctx, int32_t n_points, const tkdv_point *pts,
                                    const tkdv_plan *sigma_plans, const tkdv_mixture *mixes, const double *starts,
                                    int32_t n_user, int32_t n_starts, uint64_t seed, double margin, tkdv_plan *out,
                                    double *xhat_best, void *stream)
{
    if (!ctx) return set_err(nullptr, TKDV_E_ARG, "ctx is NULL");
    if (n_points < 0) return set_err(ctx, TKDV_E_ARG, "n_points < 0");
    if (n_points == 0) return TKDV_OK;
    if (!pts || !sigma_plans || !mixes || !out) return set_err(ctx, TKDV_E_ARG, "NULL argument");
    if (n_starts < 1 || n_starts > 256) return set_err(ctx, TKDV_E_ARG, "n_starts must be in [1, 256]");
    if (n_user < 0 || n_user > 256 || (n_user > 0 && !starts)) return set_err(ctx, TKDV_E_ARG, "bad caller starts");
    if (!(margin >= 0.0) || !std::isfinite(margin)) return set_err(ctx, TKDV_E_ARG, "margin must be >= 0");
    if ((int64_t)n_points * (n_starts + n_user) > (int64_t)(1 << 30)) return set_err(ctx, TKDV_E_ARG, "too many starts");
    std::vector<PlanPoint> pp(n_points);
    std::vector<PlanMix> pm(n_points);
    std::vector<double> user((size_t)n_points * std::max(n_user, 0) * kPlanStride, 0.0);
    std::vector<double> cap(n_points), log_eps(n_points);
    for (int p = 0; p < n_points; ++p) {
        const tkdv_point &q = pts[p];
        const tkdv_plan &sp = sigma_plans[p];
        if (q.K < 1 || q.K > 32) return set_err(ctx, TKDV_E_ARG, "point " + std::to_string(p) + ": K must be <= 32");
        if (!std::isfinite(q.E0) || !(q.E0 > 0.0) || !std::isfinite(q.beta_p) || !std::isfinite(q.c32))
            return set_err(ctx, TKDV_E_ARG, "point " + std::to_string(p) + ": bad point");
        if (sp.proposal != TKDV_PROP_SIGMA) return set_err(ctx, TKDV_E_ARG, "sigma_plans must be Sigma plans");
        MixHost mh;
        const int st = mh.init(q, sp, mixes[p]);
        if (st != TKDV_OK) return set_err(ctx, (tkdv_status)st, "point " + std::to_string(p) + ": bad mixture");
        const int K = q.K, n2 = 2 * K;
        PlanPoint P{};
        P.K = K;
        P.N = 4 * K;
        P.sigma = 0;  // log f alone; the mixture term is added in the kernel
        P.point_id = q.point_id;
        P.dt0 = -q.beta_p / ((double)K * K);
        P.cH = q.beta_p * q.c32 / (q.E0 * (double)K * K);
        const double amp = std::sqrt(2.0 * q.E0 / kPi);
        P.amp3 = amp * amp * amp;
        pp[p] = P;
        PlanMix &M = pm[p];
        std::memset(&M, 0, sizeof(M));
        for (int c = 0; c < n2; ++c) {
            M.a[c] = mh.a[c];
            M.V[c][0] = mh.V[(size_t)c * 2];
            M.V[c][1] = mh.V[(size_t)c * 2 + 1];
        }
        for (int r = 0; r < 2; ++r)
            for (int c = 0; c < 2; ++c) M.gi[r][c] = mh.Ginv[r][c];
        for (int m = 0; m < 32; ++m) {
            M.cs[m] = std::cos(2.0 * kPi * m / 32.0);
            M.sn[m] = std::sin(2.0 * kPi * m / 32.0);
        }
        M.logdetL0 = mh.logdetL0;
        M.lng = mh.lng;
        M.log_eps = mh.log_eps;
        M.log_1m_eps = mh.log_1m_eps;
        M.gc = mh.alpha * mh.beta_p / ((double)K * K * K);
        cap[p] = sp.log_M - sp.log_norm_g - mh.log_eps;
        for (int u = 0; u < n_user; ++u) {
            const double *src = starts + ((size_t)p * n_user + u) * 2 * TKDV_KMAX;
            double r2 = 0.0;
            for (int c = 0; c < n2; ++c) r2 += src[c] * src[c];
            if (!(r2 > 0.0) || !std::isfinite(r2))
                return set_err(ctx, TKDV_E_ARG, "point " + std::to_string(p) + ": a caller start is zero or not finite");
            for (int c = 0; c < n2; ++c) user[((size_t)p * n_user + u) * kPlanStride + c] = src[c];
        }
    }
    std::vector<double> val, xb;
    std::vector<int> ev;
    tkdv_status rs = run_plan_search(ctx, pp, &pm, &user, n_user, n_starts, seed, (hipStream_t)stream, val, xb, ev);
    if (rs != TKDV_OK) return rs;
    const int per = n_starts + n_user;
    for (int p = 0; p < n_points; ++p) {
        long total = 0;
        const int bi = best_item(val, ev, p, per, &total);
        if (bi < 0) return set_err(ctx, TKDV_E_DEVICE, "point " + std::to_string(p) + ": search gave no value");
        const double lm = val[bi] + std::log1p(margin);
        out[p] = sigma_plans[p];
        out[p].proposal = TKDV_PROP_MIXTURE;
        out[p].log_M = std::min(lm, cap[p]);
        out[p].M_source = lm > cap[p] ? 3 : 2;
        out[p].n_optimiser_evals = (int32_t)std::min<long>(total, INT32_MAX);
        if (xhat_best) {
            std::fill(xhat_best + (size_t)p * 2 * TKDV_KMAX, xhat_best + (size_t)(p + 1) * 2 * TKDV_KMAX, 0.0);
            for (int m = 0; m < 2 * pts[p].K; ++m) xhat_best[(size_t)p * 2 * TKDV_KMAX + m] = xb[(size_t)bi * kPlanStride + m];
        }
    }
    return TKDV_OK;
}

tkdv_status tkdv_extremes(tkdv_ctx *ctx, int32_t K, double E0, const float *d_xhat, uint64_t n, uint64_t row_stride,
                          int32_t top_k, double threshold, uint64_t *h_rows, double *h_umax, int32_t *h_jmax,
                          uint64_t *h_n_exceed, float *d_umax, int32_t *d_jmax, void *stream)
{
    if (!ctx) return set_err(nullptr, TKDV_E_ARG, "ctx is NULL");
    if (kindex(K) < 0) return set_err(ctx, TKDV_E_UNSUPPORTED, "tkdv_extremes supports K in {8,16,32,64,128}");
    if (!std::isfinite(E0) || !(E0 > 0.0)) return set_err(ctx, TKDV_E_ARG, "E0 must be finite and > 0");
    if (top_k < 0 || top_k > TKDV_EXTREMES_MAX_K) return set_err(ctx, TKDV_E_ARG, "top_k out of range");
    if (top_k > 0 && (!h_rows || !h_umax || !h_jmax)) return set_err(ctx, TKDV_E_ARG, "NULL output array");
    if (!h_n_exceed) return set_err(ctx, TKDV_E_ARG, "h_n_exceed is NULL");
    if (std::isnan(threshold)) return set_err(ctx, TKDV_E_ARG, "threshold is NaN");
    if (row_stride < (uint64_t)(2 * K) || row_stride % 4 != 0)
        return set_err(ctx, TKDV_E_ARG, "row_stride must be >= 2K and a multiple of 4");
    if (n > 0 && (!d_xhat || ((uintptr_t)d_xhat & 15u)))
        return set_err(ctx, TKDV_E_ARG, "d_xhat must be a 16-byte aligned device pointer");
    for (int i = 0; i < top_k; ++i) {
        h_rows[i] = UINT64_MAX;
        h_umax[i] = std::nan("");
        h_jmax[i] = -1;
    }
    *h_n_exceed = 0;
    if (n == 0) return TKDV_OK;
    HIP_TRY(ctx, hipSetDevice(ctx->device));
    tkdv_status bs = build_tables(ctx, K);
    if (bs != TKDV_OK) return bs;
    hipStream_t st = (hipStream_t)stream;
    const int ki = kindex(K);
    const unsigned long long cap_eq = 1ull << 16;
    const size_t k = (size_t)std::min<uint64_t>((uint64_t)top_k, n), first_eq = 64;
    HIP_TRY(ctx, ensure(ctx->ext_keys, n * sizeof(uint32_t)));
    if (!d_jmax) HIP_TRY(ctx, ensure(ctx->ext_jmax, n * sizeof(int32_t)));
    // the selection's state, then the rows above the k-th key and those equal to it;
    // its result, the former and the first of the latter are one copy
    const size_t head = offsetof(ExtSelect, out), back = sizeof(ExtSelect) - head + (k + first_eq) * sizeof(ExtRow);
    HIP_TRY(ctx, ensure(ctx->ext_misc, sizeof(ExtSelect) + (k + cap_eq) * sizeof(ExtRow)));
    HIP_TRY(ctx, ensure_host(ctx->h_misc, ctx->h_misc_bytes, back));
    ExtSelect *sel = (ExtSelect *)ctx->ext_misc.p;
    ExtRow *above = (ExtRow *)(sel + 1), *equal = above + k;
    HIP_TRY(ctx, launch_ext_begin(sel, k, st));
    ExtArgs ea{};
    ea.xhat = d_xhat;
    ea.n = n;
    ea.stride = row_stride;
    ea.phi_f32 = ki >= 3 ? ctx->qstat[ki - 3].p : ctx->phi_f32[ki].p;  // quarter-period statistics tables
    ea.amp = (float)std::sqrt(2.0 * E0 / kPi);
    ea.threshold = (float)threshold;
    ea.keys = (uint32_t *)ctx->ext_keys.p;
    ea.umax = d_umax;
    ea.jmax = d_jmax ? d_jmax : (int *)ctx->ext_jmax.p;
    ea.n_exceed = &sel->out.n_exceed;
    ea.hist = sel->hist[0];
    HIP_TRY(ctx, launch_grid_max(K, ea, ctx->n_cu, st));
    if (k > 0) HIP_TRY(ctx, launch_ext_select(ea.keys, ea.jmax, n, sel, above, k, equal, cap_eq, ctx->n_cu, st));
    char *h = (char *)ctx->h_misc;
    HIP_TRY(ctx, hipMemcpyAsync(h, (char *)sel + head, k > 0 ? back : sizeof(ExtSelect) - head, hipMemcpyDeviceToHost, st));
    HIP_TRY(ctx, hipStreamSynchronize(st));
    ExtSelect::Out out;
    std::memcpy(&out, h, sizeof(out));
    *h_n_exceed = out.n_exceed;
    if (k == 0) return TKDV_OK;
    if (out.above != k - out.need || out.equal < out.need)
        return set_err(ctx, TKDV_E_DEVICE, "tkdv_extremes: inconsistent selection counts");
    if (out.equal > cap_eq) return set_err(ctx, TKDV_E_UNSUPPORTED, "tkdv_extremes: more than 65536 tied maxima");
    const ExtRow *rows = (const ExtRow *)(h + (sizeof(ExtSelect) - head));
    std::vector<ExtRow> top(rows, rows + out.above), tied(out.equal);
    if (out.equal <= first_eq) {
        std::copy(rows + k, rows + k + out.equal, tied.begin());
    } else {
        HIP_TRY(ctx, hipMemcpyAsync(tied.data(), equal, out.equal * sizeof(ExtRow), hipMemcpyDeviceToHost, st));
        HIP_TRY(ctx, hipStreamSynchronize(st));
    }
    // larger maxima first, lower rows first among equal ones
    auto before = [](const ExtRow &x, const ExtRow &y) { return x.key != y.key ? x.key > y.key : x.row < y.row; };
    std::sort(tied.begin(), tied.end(), before);
    top.insert(top.end(), tied.begin(), tied.begin() + (std::ptrdiff_t)out.need);
    std::sort(top.begin(), top.end(), before);
    for (size_t i = 0; i < k; ++i) {
        const uint32_t bits = (top[i].key & 0x80000000u) ? (top[i].key & 0x7FFFFFFFu) : ~top[i].key;
        float f;
        std::memcpy(&f, &bits, 4);
        h_rows[i] = top[i].row;
        h_umax[i] = f;
        h_jmax[i] = top[i].j;
    }
    return TKDV_OK;
}

tkdv_status tkdv_sir(tkdv_ctx *ctx, const tkdv_point *pt, tkdv_proposal proposal, const tkdv_plan *plan, uint64_t n,
                     uint64_t m, double u0, tkdv_precision precision, uint64_t *d_index, float *d_xhat,
                     float *d_weight, tkdv_sir_stats *h_stats, void *stream)
{
    if (!ctx) return set_err(nullptr, TKDV_E_ARG, "ctx is NULL");
    if (!pt || !h_stats) return set_err(ctx, TKDV_E_ARG, "NULL argument");
    tkdv_status s = check_point(ctx, *pt);
    if (s != TKDV_OK) return s;
    if (proposal != TKDV_PROP_UNIFORM && proposal != TKDV_PROP_SIGMA)
        return set_err(ctx, TKDV_E_ARG, "proposal must be UNIFORM or SIGMA");
    if (precision != TKDV_FP32 && precision != TKDV_BF16X3)
        return set_err(ctx, TKDV_E_UNSUPPORTED, "tkdv_sir computes weights with FP32 or BF16x3 synthesis");
    if (n == 0 || n >= (1ull << 40)) return set_err(ctx, TKDV_E_ARG, "n must be in [1, 2^40)");
    if (!(u0 >= 0.0 && u0 < 1.0)) return set_err(ctx, TKDV_E_ARG, "u0 must be in [0, 1)");
    if (m > 0 && !d_index) return set_err(ctx, TKDV_E_ARG, "d_index is NULL");
    if (plan && plan->proposal != proposal) return set_err(ctx, TKDV_E_ARG, "plan is for another proposal");
    HIP_TRY(ctx, hipSetDevice(ctx->device));
    tkdv_plan pl;
    if (plan) {
        pl = *plan;
    } else {
        const int ps = plan_point_host(pt, proposal, 2, &pl);
        if (ps != TKDV_OK) return set_err(ctx, (tkdv_status)ps, "planning failed");
    }
    const int K = pt->K, ki = kindex(K);
    s = build_tables(ctx, K);
    if (s != TKDV_OK) return s;
    DevPoint d;
    fill_devpoint(d, *pt, pl, proposal, precision);
    d.i0 = 0;
    d.n = n;
    d.n_tiles = (n + kTile - 1) / kTile;
    const unsigned long long n_tiles = d.n_tiles, n_chunks = (n_tiles + kSirChunk - 1) / kSirChunk;
    const int grid = sir_grid(K, ctx->n_cu, n_tiles), waves = grid * (sir_block(K) / kWave);
    HIP_TRY(ctx, ensure(ctx->sir_pt, sizeof(DevPoint)));
    if (!d_weight) HIP_TRY(ctx, ensure(ctx->sir_w, n * sizeof(float)));
    HIP_TRY(ctx, ensure(ctx->sir_tile, 2 * n_tiles * sizeof(double)));
    HIP_TRY(ctx, ensure(ctx->sir_chunk, (2 * n_chunks + 1 + kSirPart) * sizeof(double)));
    HIP_TRY(ctx, ensure(ctx->sir_part, (size_t)waves * kSirPart * sizeof(double)));
    hipStream_t st = (hipStream_t)stream;
    HIP_TRY(ctx, hipMemcpyAsync(ctx->sir_pt.p, &d, sizeof(d), hipMemcpyHostToDevice, st));
    SirArgs a{};
    a.pt = (const DevPoint *)ctx->sir_pt.p;
    a.phi_hi = precision == TKDV_FP32 ? ctx->phi_f32[ki].p : ctx->phi_hi[ki].p;
    a.phi_lo = ctx->phi_lo[ki].p;
    a.n = n;
    a.n_tiles = n_tiles;
    a.w = d_weight ? d_weight : (float *)ctx->sir_w.p;
    a.tile_sum = (double *)ctx->sir_tile.p;
    a.tile_off = a.tile_sum + n_tiles;
    a.chunk_sum = (double *)ctx->sir_chunk.p;
    a.chunk_off = a.chunk_sum + n_chunks;
    a.sums = a.chunk_off + n_chunks + 1;
    a.n_chunks = n_chunks;
    a.waves = waves;
    a.wave_part = (double *)ctx->sir_part.p;
    a.m = m;
    a.u0 = u0;
    a.index = reinterpret_cast<unsigned long long *>(d_index);
    a.xhat = d_xhat;
    HIP_TRY(ctx, hipEventRecord(ctx->ev[0], st));
    HIP_TRY(ctx, launch_sir_weights(K, precision, proposal, a, ctx->n_cu, st));
    HIP_TRY(ctx, hipEventRecord(ctx->ev[1], st));
    HIP_TRY(ctx, launch_sir_scan(a, st));
    if (m > 0) HIP_TRY(ctx, launch_sir_resample(K, proposal, a, ctx->n_cu, st));
    HIP_TRY(ctx, hipEventRecord(ctx->ev[2], st));
    double back[1 + kSirPart];  // W and the sums over the waves
    HIP_TRY(ctx, hipMemcpyAsync(back, a.chunk_off + n_chunks, sizeof(back), hipMemcpyDeviceToHost, st));
    HIP_TRY(ctx, hipStreamSynchronize(st));
    const double W = back[0];
    if (m > 0 && !(W > 0.0)) return set_err(ctx, TKDV_E_UNSUPPORTED, "all weights are zero: nothing to resample");
    {
        float ms = 0.0f;
        ctx->timing = tkdv_timing{};
        if (hipEventElapsedTime(&ms, ctx->ev[0], ctx->ev[1]) == hipSuccess) ctx->timing.decide_ms = ms;
        if (hipEventElapsedTime(&ms, ctx->ev[0], ctx->ev[2]) == hipSuccess) ctx->timing.total_ms = ms;
        ctx->timing.decide_grid = grid;
        ctx->timing.decide_block = sir_block(K);
    }
    const double W2 = back[1], mx = back[2], *M = back + 3, over = back[7];
    std::memset(h_stats, 0, sizeof(*h_stats));
    h_stats->n = n;
    h_stats->m = m;
    h_stats->n_over_one = (uint64_t)over;
    h_stats->W = W;
    h_stats->W2 = W2;
    h_stats->ess = W2 > 0.0 ? W * W / W2 : 0.0;
    h_stats->max_w = mx;
    if (W > 0.0) {
        const double amp = std::sqrt(2.0 * pt->E0 / kPi), N = 4.0 * K;
        double ap = amp;
        double mom[4];
        for (int c = 0; c < 4; ++c, ap *= amp) mom[c] = M[c] * ap / N / W;
        h_stats->mean = mom[0];
        h_stats->m2 = mom[1];
        h_stats->m3 = mom[2];
        h_stats->m4 = mom[3];
        if (mom[1] > 0.0) {
            h_stats->skewness = mom[2] / std::pow(mom[1], 1.5);
            h_stats->kurtosis = mom[3] / (mom[1] * mom[1]);
        }
    }
    return TKDV_OK;
}

tkdv_status tkdv_sample_batch(tkdv_ctx *ctx, int32_t n_points, const tkdv_point *pts, tkdv_proposal proposal,
                              const tkdv_plan *plans, const uint64_t *n, tkdv_count_mode mode,
                              uint64_t max_proposals, tkdv_precision precision, float *d_xhat,
                              uint64_t *d_index, const uint64_t *capacity, const uint64_t *out_offset,
                              tkdv_stats *h_stats, void *stream)
{
    if (!ctx) return set_err(nullptr, TKDV_E_ARG, "ctx is NULL");
    if (!pts || !n || !h_stats) return set_err(ctx, TKDV_E_ARG, "NULL argument");
    HIP_TRY(ctx, hipSetDevice(ctx->device));
    if (n_points < 1) return set_err(ctx, TKDV_E_ARG, "n_points must be >= 1");
    std::vector<tkdv_plan> pl(n_points);
    for (int p = 0; p < n_points; ++p) {
        if (plans) {
            pl[p] = plans[p];
            continue;
        }
        tkdv_status s = check_point(ctx, pts[p]);
        if (s != TKDV_OK) return s;
        s = (tkdv_status)plan_point_host(&pts[p], proposal, 2, &pl[p]);
        if (s != TKDV_OK) return set_err(ctx, s, "planning failed");
    }
    // run every point, then again the points whose M was violated (raised M)
    std::vector<int> todo(n_points);
    for (int p = 0; p < n_points; ++p) todo[p] = p;
    for (int raise = 0; !todo.empty(); ++raise) {
        const int m = (int)todo.size();
        std::vector<tkdv_point> spt(m);
        std::vector<tkdv_plan> spl(m);
        std::vector<uint64_t> sn(m), scap(m), soff(m);
        for (int q = 0; q < m; ++q) {
            const int p = todo[q];
            spt[q] = pts[p];
            spl[q] = pl[p];
            sn[q] = n[p];
            scap[q] = capacity ? capacity[p] : 0;
            soff[q] = out_offset ? out_offset[p] : 0;
        }
        Call call;
        tkdv_status s = prepare(ctx, call, m, spt.data(), proposal, spl.data(), sn.data(), mode, max_proposals,
                                precision, scap.data(), soff.data(), 2 * TKDV_KMAX, 0);
        if (s != TKDV_OK) return s;
        std::vector<PointResult> res;
        std::vector<DevCounters> cnt;
        s = run(ctx, call, precision, proposal, d_xhat, reinterpret_cast<unsigned long long *>(d_index),
                (hipStream_t)stream, &res, &cnt, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, true);
        if (s != TKDV_OK) return s;
        std::vector<int> again;
        for (int q = 0; q < m; ++q) {
            const int p = todo[q];
            fill_stats(h_stats[p], call.pts[q], res[q], cnt[q], mode);
            h_stats[p].M_raises = raise;
            if (h_stats[p].n_M_violations == 0 || ctx->mv_policy == TKDV_MV_COUNT) continue;
            if (ctx->mv_policy == TKDV_MV_FAIL || raise == kMaxRaises) return violation_error(ctx, p, h_stats[p]);
            pl[p].log_M = raised_log_M(pl[p].log_M, h_stats[p].max_log_a, call.pts[q].tau);
            again.push_back(p);
        }
        todo.swap(again);
    }
    return TKDV_OK;
}

tkdv_status tkdv_sample(tkdv_ctx *ctx, const tkdv_point *pt, tkdv_proposal proposal, const tkdv_plan *plan,
                        uint64_t n, tkdv_count_mode mode, uint64_t max_proposals, tkdv_precision precision,
                        float *d_xhat, uint64_t *d_index, uint64_t capacity, tkdv_stats *h_stats, void *stream)
{
    if (!ctx) return set_err(nullptr, TKDV_E_ARG, "ctx is NULL");
    if (!pt || !h_stats) return set_err(ctx, TKDV_E_ARG, "NULL argument");
    HIP_TRY(ctx, hipSetDevice(ctx->device));
    if (n == 0) {
        std::memset(h_stats, 0, sizeof(*h_stats));
        tkdv_status s = check_point(ctx, *pt);
        if (s != TKDV_OK) return s;
        const double umax = std::sqrt(2.0 * pt->K * pt->E0 / kPi);
        h_stats->hist_lo = -umax;
        h_stats->hist_hi = umax;
        h_stats->max_log_a = -INFINITY;
        h_stats->log_M_used = plan ? plan->log_M : NAN;
        return TKDV_OK;
    }
    tkdv_plan pl;
    if (plan) {
        pl = *plan;
    } else {
        tkdv_status s = check_point(ctx, *pt);
        if (s != TKDV_OK) return s;
        s = (tkdv_status)plan_point_host(pt, proposal, 2, &pl);
        if (s != TKDV_OK) return set_err(ctx, s, "planning failed");
    }
    for (int raise = 0;; ++raise) {
        Call call;
        const uint64_t cap = capacity, off = 0;
        tkdv_status s = prepare(ctx, call, 1, pt, proposal, &pl, &n, mode, max_proposals, precision, &cap, &off,
                                2 * (uint64_t)pt->K, 0);
        if (s != TKDV_OK) return s;
        std::vector<PointResult> res;
        std::vector<DevCounters> cnt;
        s = run(ctx, call, precision, proposal, d_xhat, reinterpret_cast<unsigned long long *>(d_index),
                (hipStream_t)stream, &res, &cnt, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, true);
        if (s != TKDV_OK) return s;
        fill_stats(*h_stats, call.pts[0], res[0], cnt[0], mode);
        h_stats->M_raises = raise;
        if (h_stats->n_M_violations == 0 || ctx->mv_policy == TKDV_MV_COUNT) return TKDV_OK;
        if (ctx->mv_policy == TKDV_MV_FAIL || raise == kMaxRaises) return violation_error(ctx, 0, *h_stats);
        pl.log_M = raised_log_M(pl.log_M, h_stats->max_log_a, call.pts[0].tau);
    }
}

tkdv_status tkdv_eval_proposals(tkdv_ctx *ctx, const tkdv_point *pt, tkdv_proposal proposal, const tkdv_plan *plan,
                                uint64_t i0, uint64_t n, tkdv_precision precision, float *d_xhat, float *d_t,
                                float *d_s3, float *d_log_a, float *d_log_u, uint8_t *d_accept, void *stream)
{
    if (!ctx) return set_err(nullptr, TKDV_E_ARG, "ctx is NULL");
    if (!pt) return set_err(ctx, TKDV_E_ARG, "NULL argument");
    if (n == 0) return TKDV_OK;
    const int any_dbg = (d_t != nullptr) + (d_s3 != nullptr) + (d_log_a != nullptr) + (d_log_u != nullptr);
    if (any_dbg != 0 && any_dbg != 4)
        return set_err(ctx, TKDV_E_ARG, "d_t, d_s3, d_log_a and d_log_u must be all set or all NULL");
    HIP_TRY(ctx, hipSetDevice(ctx->device));
    Call call;
    const uint64_t zero = 0;
    tkdv_status s = prepare(ctx, call, 1, pt, proposal, plan, &n, TKDV_COUNT_PROPOSALS, 0, precision, &zero, &zero,
                            2 * (uint64_t)pt->K, i0);
    if (s != TKDV_OK) return s;
    s = run(ctx, call, precision, proposal, nullptr, nullptr, (hipStream_t)stream, nullptr, nullptr, nullptr, d_xhat,
            d_t, d_s3, d_log_a, d_log_u, false);
    if (s != TKDV_OK) return s;
    if (d_accept) {
        HIP_TRY(ctx, launch_bits_to_bytes(reinterpret_cast<const uint32_t *>(ctx->bitmap.p), n, d_accept,
                                          (hipStream_t)stream));
        HIP_TRY(ctx, hipStreamSynchronize((hipStream_t)stream));
    }
    return TKDV_OK;
}

tkdv_status tkdv_sample_mixture(tkdv_ctx *ctx, const tkdv_point *pt, const tkdv_plan *mix_plan,
                                const tkdv_mixture *mix, uint64_t n, tkdv_count_mode mode,
                                uint64_t max_proposals, tkdv_precision precision, float *d_xhat,
                                uint64_t *d_index, uint64_t capacity, tkdv_stats *h_stats, void *stream)
{
    if (!ctx) return set_err(nullptr, TKDV_E_ARG, "ctx is NULL");
    if (!pt || !h_stats || !mix_plan || !mix) return set_err(ctx, TKDV_E_ARG, "NULL argument");
    HIP_TRY(ctx, hipSetDevice(ctx->device));
    if (n == 0) {
        std::memset(h_stats, 0, sizeof(*h_stats));
        tkdv_status s = check_point(ctx, *pt);
        if (s != TKDV_OK) return s;
        const double umax = std::sqrt(2.0 * pt->K * pt->E0 / kPi);
        h_stats->hist_lo = -umax;
        h_stats->hist_hi = umax;
        h_stats->max_log_a = -INFINITY;
        h_stats->log_M_used = mix_plan->log_M;
        return TKDV_OK;
    }
    hipStream_t st = (hipStream_t)stream;
    tkdv_plan pl = *mix_plan;
    for (int raise = 0; raise <= kMaxRaises; ++raise) {
        Call call;
        const uint64_t cap = capacity, off = 0;
        tkdv_status s = prepare(ctx, call, 1, pt, TKDV_PROP_MIXTURE, &pl, &n, mode, max_proposals, precision, &cap,
                                &off, 2 * (uint64_t)pt->K, 0);
        if (s != TKDV_OK) return s;
        s = prepare_mixture(ctx, call, *pt, pl, mix, precision, st);
        if (s != TKDV_OK) return s;
        std::vector<PointResult> res;
        std::vector<DevCounters> cnt;
        s = run(ctx, call, precision, TKDV_PROP_MIXTURE, d_xhat, reinterpret_cast<unsigned long long *>(d_index),
                st, &res, &cnt, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, true);
        if (s != TKDV_OK) return s;
        fill_stats(*h_stats, call.pts[0], res[0], cnt[0], mode);
        h_stats->M_raises = raise;
        if (h_stats->n_M_violations == 0 || ctx->mv_policy == TKDV_MV_COUNT) return TKDV_OK;
        if (ctx->mv_policy == TKDV_MV_FAIL) return violation_error(ctx, 0, *h_stats);
        pl.log_M = raised_log_M(pl.log_M, h_stats->max_log_a, call.pts[0].tau);
    }
    // the mixture's bound kept failing: the paper's Sigma sampler (itself
    // guarded the same way) produces the exact samples instead
    tkdv_plan sp;
    tkdv_status s = (tkdv_status)plan_point_host(pt, TKDV_PROP_SIGMA, 2, &sp);
    if (s != TKDV_OK) return set_err(ctx, s, "planning the Sigma fallback failed");
    s = tkdv_sample(ctx, pt, TKDV_PROP_SIGMA, &sp, n, mode, max_proposals, precision, d_xhat, d_index, capacity,
                    h_stats, stream);
    if (s != TKDV_OK) return s;
    h_stats->fallback = 1;
    return TKDV_OK;
}

tkdv_status tkdv_eval_mixture(tkdv_ctx *ctx, const tkdv_point *pt, const tkdv_plan *mix_plan,
                              const tkdv_mixture *mix, uint64_t i0, uint64_t n, tkdv_precision precision,
                              float *d_xhat, float *d_t, float *d_s3, float *d_log_a, float *d_log_u,
                              uint8_t *d_accept, void *stream)
{
    if (!ctx) return set_err(nullptr, TKDV_E_ARG, "ctx is NULL");
    if (!pt || !mix_plan || !mix) return set_err(ctx, TKDV_E_ARG, "NULL argument");
    if (n == 0) return TKDV_OK;
    const int any_dbg = (d_t != nullptr) + (d_s3 != nullptr) + (d_log_a != nullptr) + (d_log_u != nullptr);
    if (any_dbg != 0 && any_dbg != 4)
        return set_err(ctx, TKDV_E_ARG, "d_t, d_s3, d_log_a and d_log_u must be all set or all NULL");
    HIP_TRY(ctx, hipSetDevice(ctx->device));
    Call call;
    const uint64_t zero = 0;
    tkdv_status s = prepare(ctx, call, 1, pt, TKDV_PROP_MIXTURE, mix_plan, &n, TKDV_COUNT_PROPOSALS, 0, precision,
                            &zero, &zero, 2 * (uint64_t)pt->K, i0);
    if (s != TKDV_OK) return s;
    hipStream_t st = (hipStream_t)stream;
    s = prepare_mixture(ctx, call, *pt, *mix_plan, mix, precision, st);
    if (s != TKDV_OK) return s;
    s = run(ctx, call, precision, TKDV_PROP_MIXTURE, nullptr, nullptr, st, nullptr, nullptr, nullptr, d_xhat, d_t,
            d_s3, d_log_a, d_log_u, false);
    if (s != TKDV_OK) return s;
    if (d_accept) {
        HIP_TRY(ctx, launch_bits_to_bytes(reinterpret_cast<const uint32_t *>(ctx->bitmap.p), n, d_accept, st));
        HIP_TRY(ctx, hipStreamSynchronize(st));
    }
    return TKDV_OK;
}

double tkdv_mixture_window(const tkdv_point *pt, const tkdv_plan *mix_plan, const tkdv_mixture *mix,
                           tkdv_precision precision)
{
    if (!pt || !mix_plan || !mix) return NAN;
    MixHost mh;
    if (mh.init(*pt, *mix_plan, *mix) != TKDV_OK) return NAN;
    return window(*pt, TKDV_PROP_MIXTURE, precision, mix_plan->alpha_star, mix_plan->log_M,
                  mix_window_extra(mh, precision));
}

double tkdv_decision_window(const tkdv_point *pt, tkdv_proposal proposal, tkdv_precision precision)
{
    if (!pt) return NAN;
    tkdv_plan pl;
    if (plan_point_host(pt, proposal, 2, &pl) != TKDV_OK) return NAN;
    return window(*pt, proposal, precision, pl.alpha_star, pl.log_M);
}

tkdv_status tkdv_synthesize(tkdv_ctx *ctx, int32_t K, tkdv_precision precision, const float *d_xhat, uint64_t n,
                            float *d_s3, void *stream)
{
    if (!ctx) return set_err(nullptr, TKDV_E_ARG, "ctx is NULL");
    if (kindex(K) < 0) return set_err(ctx, TKDV_E_UNSUPPORTED, "tkdv_synthesize supports K in {8,16,32,64,128}");
    if (precision < TKDV_FP32 || precision > TKDV_BF16X3) return set_err(ctx, TKDV_E_ARG, "bad precision");
    if (n == 0) return TKDV_OK;
    if (!d_xhat || !d_s3) return set_err(ctx, TKDV_E_ARG, "NULL device pointer");
    if ((uintptr_t)d_xhat & 15u) return set_err(ctx, TKDV_E_ARG, "d_xhat must be 16-byte aligned");
    HIP_TRY(ctx, hipSetDevice(ctx->device));
    tkdv_status s = build_tables(ctx, K);
    if (s != TKDV_OK) return s;
    const int ki = kindex(K);
    hipStream_t st = (hipStream_t)stream;
    std::memset(&ctx->timing, 0, sizeof(ctx->timing));
    const void *tab_hi = nullptr, *tab_lo = nullptr;
    s3_tables(ctx, ki, precision, tab_hi, tab_lo);
    auto launch = K == 128 ? launch_synth_quarter : launch_synth;
    HIP_TRY(ctx, launch(K, precision, d_xhat, n, d_s3, tab_hi, tab_lo, ctx->n_cu, st, ctx->ev[0],
                        &ctx->timing.decide_grid, &ctx->timing.decide_block));
    HIP_TRY(ctx, hipEventRecord(ctx->ev[1], st));
    HIP_TRY(ctx, hipEventSynchronize(ctx->ev[1]));
    float ms = 0.0f;
    HIP_TRY(ctx, hipEventElapsedTime(&ms, ctx->ev[0], ctx->ev[1]));
    ctx->timing.synth_ms = ms;
    ctx->timing.total_ms = ms;
    return TKDV_OK;
}

tkdv_status tkdv_sample_sweep(tkdv_ctx *ctx, int32_t n_points, const tkdv_point *pts, const tkdv_plan *plans,
                              const uint64_t *targets, const uint64_t *max_proposals, tkdv_precision precision,
                              const tkdv_launch_cfg *cfg, float *d_xhat, uint64_t *d_index,
                              const uint64_t *capacity, const uint64_t *out_offset, tkdv_stats *h_stats,
                              void *stream)
{
    if (!ctx) return set_err(nullptr, TKDV_E_ARG, "ctx is NULL");
    HIP_TRY(ctx, hipSetDevice(ctx->device));
    if (n_points < 1 || !pts || !targets || !max_proposals || !h_stats)
        return set_err(ctx, TKDV_E_ARG, "n_points must be >= 1 and the arrays non-NULL");
    std::vector<tkdv_plan> pl(n_points);
    for (int p = 0; p < n_points; ++p) {
        if (plans) {
            pl[p] = plans[p];
            continue;
        }
        tkdv_status s = check_point(ctx, pts[p]);
        if (s != TKDV_OK) return s;
        s = (tkdv_status)plan_point_host(&pts[p], TKDV_PROP_SIGMA, 2, &pl[p]);
        if (s != TKDV_OK) return set_err(ctx, s, "planning failed");
    }
    std::vector<int> todo(n_points);
    for (int p = 0; p < n_points; ++p) todo[p] = p;
    for (int raise = 0; !todo.empty(); ++raise) {
        const int m = (int)todo.size();
        std::vector<tkdv_point> spt(m);
        std::vector<tkdv_plan> spl(m);
        std::vector<uint64_t> stg(m), smax(m), scap(m), soff(m);
        std::vector<tkdv_stats> sst(m);
        for (int q = 0; q < m; ++q) {
            const int p = todo[q];
            spt[q] = pts[p];
            spl[q] = pl[p];
            stg[q] = targets[p];
            smax[q] = max_proposals[p];
            scap[q] = capacity ? capacity[p] : 0;
            soff[q] = out_offset ? out_offset[p] : 0;
        }
        tkdv_status s = sweep(ctx, m, spt.data(), spl.data(), stg.data(), smax.data(), precision, cfg, d_xhat,
                              d_index, scap.data(), soff.data(), sst.data(), (hipStream_t)stream);
        if (s != TKDV_OK) return s;
        std::vector<int> again;
        for (int q = 0; q < m; ++q) {
            const int p = todo[q];
            h_stats[p] = sst[q];
            h_stats[p].M_raises = raise;
            if (sst[q].n_M_violations == 0 || ctx->mv_policy == TKDV_MV_COUNT) continue;
            if (ctx->mv_policy == TKDV_MV_FAIL || raise == kMaxRaises) return violation_error(ctx, p, sst[q]);
            pl[p].log_M = raised_log_M(pl[p].log_M, sst[q].max_log_a, window(pts[p], TKDV_PROP_SIGMA, precision,
                                                                             pl[p].alpha_star, pl[p].log_M));
            again.push_back(p);
        }
        todo.swap(again);
    }
    return TKDV_OK;
}

tkdv_status tkdv_extremes_map(tkdv_ctx *ctx, int32_t K, double E0, int32_t n_beta, const double *betas,
                              int32_t n_c, const double *c32s, uint64_t seed, uint32_t point_id0,
                              uint64_t n_accepted, uint64_t max_proposals, tkdv_precision precision,
                              tkdv_map_cell *cells, void *stream)
{
    if (!ctx) return set_err(nullptr, TKDV_E_ARG, "ctx is NULL");
    if (!betas || !c32s || !cells) return set_err(ctx, TKDV_E_ARG, "NULL argument");
    if (n_beta < 1 || n_c < 1 || (int64_t)n_beta * n_c > TKDV_MAP_MAX_CELLS)
        return set_err(ctx, TKDV_E_ARG, "n_beta, n_c >= 1 and n_beta * n_c <= TKDV_MAP_MAX_CELLS");
    if (n_accepted < 1 || max_proposals < 1) return set_err(ctx, TKDV_E_ARG, "n_accepted, max_proposals >= 1");
    if (precision != TKDV_FP32 && precision != TKDV_BF16X3)
        return set_err(ctx, TKDV_E_UNSUPPORTED, "the map decides with FP32 or BF16x3 products");
    std::vector<tkdv_point> pts;
    std::vector<int> cell_of;
    for (int b = 0; b < n_beta; ++b)
        for (int c = 0; c < n_c; ++c) {
            const int q = b * n_c + c;
            tkdv_map_cell &m = cells[q];
            std::memset(&m, 0, sizeof(m));
            m.beta_p = betas[b];
            m.c32 = c32s[c];
            m.peak_u = -INFINITY;
            m.peak_index = UINT64_MAX;
            tkdv_point pt;
            std::memset(&pt, 0, sizeof(pt));
            pt.K = K;
            pt.point_id = point_id0 + (uint32_t)q;
            pt.E0 = E0;
            pt.beta_p = betas[b];
            pt.c32 = c32s[c];
            pt.seed = seed;
            tkdv_status s = check_point(ctx, pt);
            if (s != TKDV_OK) return s;
            double alpha = 0.0;
            const int rs = plan_alpha_star(K, pt.beta_p, &alpha);
            if (rs == TKDV_E_NO_ALPHA_ROOT) {
                m.status = TKDV_E_NO_ALPHA_ROOT;
                continue;
            }
            if (rs != TKDV_OK) return set_err(ctx, (tkdv_status)rs, "bad beta'");
            pts.push_back(pt);
            cell_of.push_back(q);
        }
    const int np = (int)pts.size();
    if (np == 0) return TKDV_OK;
    std::vector<tkdv_plan> plans(np);
    tkdv_status s = tkdv_plan_batch(ctx, np, pts.data(), TKDV_PROP_SIGMA, 16, seed, 0, plans.data(), nullptr, stream);
    if (s != TKDV_OK) return s;
    std::vector<uint64_t> targets(np, n_accepted), maxp(np, max_proposals);
    std::vector<tkdv_stats> st(np);
    s = tkdv_sample_sweep(ctx, np, pts.data(), plans.data(), targets.data(), maxp.data(), precision, nullptr,
                          nullptr, nullptr, nullptr, nullptr, st.data(), stream);
    if (s != TKDV_OK) return s;
    for (int q = 0; q < np; ++q) {
        tkdv_map_cell &m = cells[cell_of[q]];
        const tkdv_stats &r = st[q];
        m.alpha_star = plans[q].alpha_star;
        m.log_M = r.log_M_used;
        m.n_proposed = r.n_proposed;
        m.n_accepted = r.n_accepted;
        m.acceptance = r.n_proposed ? (double)r.n_accepted / (double)r.n_proposed : 0.0;
        m.skewness = r.skewness;
        m.kurtosis = r.kurtosis;
        m.p_exceed_2sigma = r.p_exceed_2sigma;
        m.p_exceed_4sigma = r.n_grid_values ? (double)r.n_exceed_4sigma / (double)r.n_grid_values : 0.0;
        m.p_sample_4sigma = r.n_accepted ? (double)r.n_samples_4sigma / (double)r.n_accepted : 0.0;
        m.peak_u = r.peak_u;
        m.peak_index = r.peak_index;
        m.M_raises = r.M_raises;
        m.status = TKDV_OK;
    }
    return TKDV_OK;
}

tkdv_status tkdv_set_violation_policy(tkdv_ctx *ctx, tkdv_violation_policy policy)
{
    if (!ctx) return set_err(nullptr, TKDV_E_ARG, "ctx is NULL");
    if (policy != TKDV_MV_RAISE && policy != TKDV_MV_FAIL && policy != TKDV_MV_COUNT)
        return set_err(ctx, TKDV_E_ARG, "bad violation policy");
    ctx->mv_policy = policy;
    return TKDV_OK;
}

tkdv_status tkdv_set_launch_cfg(tkdv_ctx *ctx, int32_t K, tkdv_precision precision, const tkdv_launch_cfg *cfg)
{
    if (!ctx || !cfg) return set_err(nullptr, TKDV_E_ARG, "NULL argument");
    if (kindex(K) < 0 || precision < TKDV_FP32 || precision > TKDV_BF16X3)
        return set_err(ctx, TKDV_E_ARG, "bad K or precision");
    if (precision == TKDV_BF16) return set_err(ctx, TKDV_E_UNSUPPORTED, kBf16Refused);
    if (cfg->window < 65536 || cfg->window % 65536 != 0 || cfg->window > (1ull << 34) || cfg->blocks_per_cu < 0 ||
        cfg->variant < 0 || cfg->variant >= TKDV_DECIDE_VARIANTS || (cfg->adaptive != 0 && cfg->adaptive != 1))
        return set_err(ctx, TKDV_E_ARG,
                       "window must be a multiple of 65536 in [65536, 2^34], variant in [0, 4), adaptive 0 or 1");
    ctx->lcfg[kindex(K)][precision] = *cfg;
    return TKDV_OK;
}

tkdv_status tkdv_get_launch_cfg(const tkdv_ctx *ctx, int32_t K, tkdv_precision precision, tkdv_launch_cfg *out)
{
    if (!ctx || !out) return set_err(nullptr, TKDV_E_ARG, "NULL argument");
    if (kindex(K) < 0 || precision < TKDV_FP32 || precision > TKDV_BF16X3)
        return set_err(nullptr, TKDV_E_ARG, "bad K or precision");
    *out = ctx->lcfg[kindex(K)][precision];
    return TKDV_OK;
}

tkdv_status tkdv_autotune(tkdv_ctx *ctx, int32_t K, tkdv_precision precision, const char *cache_path,
                          tkdv_launch_cfg *out)
{
    if (!ctx) return set_err(nullptr, TKDV_E_ARG, "ctx is NULL");
    if (kindex(K) < 0 || precision < TKDV_FP32 || precision > TKDV_BF16X3)
        return set_err(ctx, TKDV_E_ARG, "bad K or precision");
    if (precision == TKDV_BF16) return set_err(ctx, TKDV_E_UNSUPPORTED, kBf16Refused);
    HIP_TRY(ctx, hipSetDevice(ctx->device));
    char key[160];
    std::snprintf(key, sizeof(key), "%s:%d K=%d prec=%d", ctx->arch.c_str(), ctx->n_cu, K, (int)precision);
    if (cache_path) {
        if (FILE *f = std::fopen(cache_path, "r")) {
            char line[512];
            while (std::fgets(line, sizeof(line), f)) {
                const size_t kl = std::strlen(key);
                if (std::strncmp(line, key, kl) != 0 || line[kl] != ' ') continue;
                int bpc = 0, graph = 1, var = 0, adap = 1;
                unsigned long long win = 0;
                if (std::sscanf(line + kl, " bpc=%d window=%llu graph=%d variant=%d adaptive=%d", &bpc, &win, &graph,
                                &var, &adap) == 5 &&
                    win >= 65536 && win % 65536 == 0 && bpc >= 0 && var >= 0 && var < TKDV_DECIDE_VARIANTS) {
                    std::fclose(f);
                    tkdv_launch_cfg c{bpc, graph, win, var, adap};
                    ctx->lcfg[kindex(K)][precision] = c;
                    if (out) *out = c;
                    return TKDV_OK;
                }
            }
            std::fclose(f);
        }
    }
    // probe: 16 points of this K, beta' in [20, 60], beta'C3/C2 = 6000 (K/32)^2,
    // a fixed number of proposals each (the targets are never met), fixed windows
    const int np = 16;
    const uint64_t per_point = K >= 64 ? (1ull << 26) : (1ull << 27);
    std::vector<tkdv_point> pts(np);
    std::vector<tkdv_plan> plans(np);
    std::vector<uint64_t> tgt(np, ~0ull >> 24), maxp(np, per_point), cap(np, 0), off(np, 0);
    for (int p = 0; p < np; ++p) {
        const double bp = 20.0 + 40.0 * p / (np - 1);
        pts[p] = tkdv_point{K, (uint32_t)p, 1.0, bp, 6000.0 * (K / 32.0) * (K / 32.0) / bp, 1234567ull + p};
    }
    if (tkdv_plan_batch(ctx, np, pts.data(), TKDV_PROP_SIGMA, 16, 7, 0, plans.data(), nullptr, nullptr) != TKDV_OK)
        return set_err(ctx, TKDV_E_DEVICE, "autotune planning failed: " + ctx->last_error);
    std::vector<tkdv_stats> st(np);
    tkdv_launch_cfg best{0, 1, 1ull << 26, 0, 1};
    double best_rate = -1.0;
    const uint64_t windows[3] = {1ull << 24, 1ull << 25, 1ull << 26};
    const int n_var = decide_n_variants(K, precision);
    for (int var = 0; var < n_var; ++var) {
        const int max_bpc = decide_variant_max_blocks_per_cu(K, precision, var);
        for (int bpc = 1; bpc <= max_bpc; ++bpc)
            for (uint64_t w : windows) {
                tkdv_launch_cfg c{bpc, 1, w, var, 0};
                tkdv_status s = sweep(ctx, np, pts.data(), plans.data(), tgt.data(), maxp.data(), precision, &c,
                                      nullptr, nullptr, cap.data(), off.data(), st.data(), nullptr);
                if (s != TKDV_OK) return s;
                const double rate = (double)per_point * np / (ctx->timing.total_ms * 1e-3);
                if (rate > best_rate) {
                    best_rate = rate;
                    best = c;
                }
            }
    }
    best.adaptive = 1;  // the probe runs fixed windows; sweeps size later windows adaptively
    ctx->lcfg[kindex(K)][precision] = best;
    if (out) *out = best;
    if (cache_path) {
        if (FILE *f = std::fopen(cache_path, "a")) {
            std::fprintf(f, "%s bpc=%d window=%llu graph=%d variant=%d adaptive=%d rate=%.6e\n", key,
                         best.blocks_per_cu, (unsigned long long)best.window, best.use_graph, best.variant,
                         best.adaptive, best_rate);
            std::fclose(f);
        }
    }
    return TKDV_OK;
}

tkdv_status tkdv_get_timing(const tkdv_ctx *ctx, tkdv_timing *out)
{
    if (!ctx || !out) return set_err(nullptr, TKDV_E_ARG, "NULL argument");
    *out = ctx->timing;
    return TKDV_OK;
}

const char *tkdv_status_str(tkdv_status s)
{
    switch (s) {
    case TKDV_OK: return "ok";
    case TKDV_E_ARG: return "invalid argument";
    case TKDV_E_NO_ALPHA_ROOT: return "F(alpha) has no root for this (K, beta')";
    case TKDV_E_DEVICE: return "HIP error";
    case TKDV_E_CAPACITY: return "internal list capacity exceeded";
    case TKDV_E_UNSUPPORTED: return "unsupported K for the GPU path";
    case TKDV_E_M_VIOLATION: return "rejection constant violated";
    }
    return "unknown status";
}

const char *tkdv_last_error(const tkdv_ctx *ctx)
{
    if (ctx) return ctx->last_error.c_str();
    std::lock_guard<std::mutex> g(g_err_mu);
    return g_last_error.c_str();
}

}  // extern "C"
