// gfx950 kernels of the TKdV rejection sampler.
//
// Pipeline of one sampling call (all on one stream, no host round trip):
//   k_decide       per wave, tiles of 32 proposals dealt out evenly or claimed
//                  from a per-point queue; Philox -> Box-Muller -> scale ->
//                  project -> t, matrix-core synthesis -> sum u^3 -> log a ->
//                  decision, two tiles at once.
//                  Writes one accept-bit word per tile; proposals within the
//                  decision window go to the FP64 list.
//   k_fixup        FP64 re-decision of the listed proposals (H3 by the double
//                  sum of Sec. IV.A), OR-ed into the accept bitmap; lays out
//                  the segments of the ordered output.
//   k_seg_count    accepted count per segment.
//   k_seg_scan     exclusive scan of the segment counts; the runs of ranks.
//   k_materialize  a wave per run of ranks: the accepted proposals in order,
//                  queued in LDS; regenerates each accepted x^ (same
//                  arithmetic as k_decide), writes it at its rank, and
//                  accumulates FP64 moments, 2-sigma exceedances and the u(0)
//                  histogram from an FP32 matrix-core synthesis.
//   k_finalize     per point, the runs' partials summed in a fixed order.
//   (mixture)      k_decide_mix and k_fixup_mix take the places of k_decide
//                  and k_fixup for the learned proposal.
#include <hip/hip_runtime.h>

#include "tkdv_device.h"
#include "tkdv_kernels.h"

namespace tkdv {

static_assert(kClaimTiles == kWave, "one accept word per lane per claim");

// k_decide's synthesis form: the half-period form (half the matrix work and
// half the tables) where it is faster, the plain product elsewhere
template <int K>
__host__ __device__ constexpr bool decide_half_period() { return K >= 16; }

// k_decide: one staged table (hi or lo)
template <int K, int PREC>
__host__ __device__ constexpr int decide_tab_bytes()
{
    return decide_half_period<K>() ? eo_table_bytes<K, PREC>()
                                   : (PREC == PREC_FP32 ? f32_table_bytes<K>() : bf16_table_bytes<K>());
}
template <int K, int PREC>
__host__ __device__ constexpr int decide_lds_bytes()
{
    return (PREC == PREC_BF16X3 ? 2 : 1) * decide_tab_bytes<K, PREC>();
}

// ---------------------------------------------------------------------------
// k_decide
// ---------------------------------------------------------------------------
// B threads per workgroup sharing one copy of the tables; G tile pairs of the
// half-period synthesis with their accumulators live together (a tile variant
// the sweep's autotuner chooses among; G divides the K/16 tile pairs).  At K = 16
// two registers more than the 128 of four waves per SIMD would leave three.
template <int K, int PREC, int PROP, int B = decide_block(K), int G = 1>
__global__ void __launch_bounds__(B, K <= 16 ? 4 : 1) k_decide(KernelArgs a, const int *plist, int n_plist)
{
    static_assert(K < 16 || (K / 16) % G == 0, "G must divide the tile pairs");
    if (a.d_active && *a.d_active == 0ull) return;  // a sweep window without unfinished points
    extern __shared__ __attribute__((aligned(16))) char lds[];
    __shared__ DeferList deferred;
    deferred.begin();
    constexpr int tab = decide_tab_bytes<K, PREC>();
    if constexpr (!decide_half_period<K>()) {
        const uint4 *s0 = reinterpret_cast<const uint4 *>(a.phi_hi);
        uint4 *d = reinterpret_cast<uint4 *>(lds);
        for (int v = threadIdx.x; v < tab / 16; v += B) d[v] = s0[v];
        if constexpr (PREC == PREC_BF16X3) {
            const uint4 *s1 = reinterpret_cast<const uint4 *>(a.phi_lo);
            for (int v = threadIdx.x; v < tab / 16; v += B) d[tab / 16 + v] = s1[v];
        }
    } else {
        stage_eo_tables<K, PREC, B>(lds, a.phi_hi, a.phi_lo);
    }
    __syncthreads();
    const char *lds_hi = lds;
    const char *lds_lo = lds + tab;
    const int lane = threadIdx.x & 63, half = lane >> 5, pl = lane & 31;
    const unsigned gwave = __builtin_amdgcn_readfirstlane(blockIdx.x * (B / kWave) + (threadIdx.x >> 6));
    const unsigned W = gridDim.x * (B / kWave);
    const float share = (float)n_plist / (2.0f * (float)W);
    PointTally tally;
    const PairCarry<3> carry{reinterpret_cast<float *>(lds + decide_lds_bytes<K, PREC>()) +
                             (threadIdx.x >> 6) * (PairCarry<3>::BYTES / 4)};
    WaveWork<K> work(gwave, n_plist);
    unsigned long long base;
    int len;
    while (work.next(a, plist, n_plist, gwave, W, share, lane, tally, base, len)) {
        const int p = __builtin_amdgcn_readfirstlane(work.p);
        const DevPoint &P = a.pts[p];
        DevCounters *C = a.cnt + p;
        // accept bits and FP64 bits of tile `lane` of this claim
        uint32_t my_word = 0u, my_def = 0u;
        const int len2 = (len + 1) & ~1;
        const unsigned long long stop = claim_stop(P, base, len);
#pragma unroll 1
        for (int c = 0; c < len2; ++c) {
            // the point's constants stay in memory from tile to tile: hoisted out
            // of this loop they would take K registers a lane
            asm volatile("" ::: "memory");
            const unsigned long long tile = base + c;
            float x[K], r2, tk;
            // x is not projected: the cube sum of u~' = Phi^T x is scaled by |x|^-3
            gen_x_part<K, PROP, true>(P, P.i0 + tile * kTile + pl, half, x, r2, tk);
            if (a.dbg_xhat) {
                const float inv = __builtin_amdgcn_rsqf(sum32(r2));
                const unsigned long long local = tile * kTile + pl;
                if (local < stop) {
#pragma unroll
                    for (int j = 0; j < K; ++j) a.dbg_xhat[local * (2 * K) + half * K + j] = x[j] * inv;
                }
            }
            float s3l;
            if constexpr (decide_half_period<K>()) s3l = eo_cube_sum<K, PREC, G>(x, lds_hi, lds_lo, lane);
            else s3l = synth_cube_sum<K, PREC>(x, lds_hi, lds_lo, lane);
            carry.put(0, c & 1, lane, r2);
            carry.put(1, c & 1, lane, tk);
            carry.put(2, c & 1, lane, s3l);
            if ((c & 1) == 0) continue;
            // settle both tiles at once, a proposal per lane: lane l takes proposal
            // 32 (c - 1) + l of the claim (one acceptance word, log a and verdict for
            // each proposal instead of two).  1e9 proposals at K = 32: 46.8 -> 45.2 ms; 2e7 at
            // K = 16 in FP32: 800 -> 752 us
            wave_lds_sync();
            const float inv = __builtin_amdgcn_rsqf(carry.sum(0, half, pl));
            const float t = carry.sum(1, half, pl) * (inv * inv);
            const float s3 = carry.sum(2, half, pl) * (inv * inv * inv);
            wave_lds_sync();
            const unsigned long long local = (tile - 1) * kTile + lane;
            const bool valid = local < stop;
            const uint32_t w_acc = acceptance_word<K>(P, P.i0 + local);
            const float la = log_a_f32<PROP>(P, t, s3);
            bool accept, defer;
            verdict(P, la, w_acc, valid, accept, defer);
            const unsigned long long bacc = __ballot(accept);
            const unsigned long long bdef = __ballot(defer);
            if ((lane | 1) == c) my_word = (uint32_t)((lane & 1) ? bacc >> 32 : bacc);
            if (bdef) {
                if ((lane | 1) == c) my_def = (uint32_t)((lane & 1) ? bdef >> 32 : bdef);
            }
            if (valid) {
                // window proposals are counted by their FP64 value (k_fixup)
                tally.n_viol += (la > 0.0f && !defer) ? 1u : 0u;
                tally.max_la = fmaxf(tally.max_la, la);
                if (a.dbg_t) {
                    a.dbg_t[local] = t;
                    a.dbg_s3[local] = s3;
                    a.dbg_log_a[local] = la;
                    a.dbg_log_u[local] = log_u_word(w_acc);
                }
            }
        }
        // one coalesced store of the claim's accept words
        if (lane < len) a.bitmap[P.bm_off + base + lane] = my_word;
        deferred.push(a, C, p, P.i0 + base * kTile, my_def, lane);
        count_accepted(P, C, my_word, len, lane);
    }
    deferred.flush(a);
}

// ---------------------------------------------------------------------------
// k_decide_mix: the sampler with the learned mixture proposal.  Workgroups
// visit the points in turn (starting at their own index) and stage the
// point's shift tables in LDS next to the synthesis tables; the waves of a
// workgroup claim tiles of that point until its queue is empty.  Per
// proposal, on top of the paper's steps: the component draw, y = (R_j A V)^T X
// for the S shifts on the matrix cores and log q_mix (mix_log_q_f32).
// ---------------------------------------------------------------------------
template <int K, int PREC>
__host__ __device__ constexpr int mix_ytab_lds_bytes()
{
    return PREC == PREC_FP32 ? mix_ytab_f32_bytes<K>() : (PREC == PREC_BF16X3 ? 2 : 1) * mix_ytab_bf16_bytes<K>();
}
// the mixture kernel's synthesis form and its tables (hi and lo) in LDS
template <int K>
__host__ __device__ constexpr bool mix_half_period() { return K >= 16; }
template <int K, int PREC>
__host__ __device__ constexpr int mix_tab_bytes()
{
    return mix_half_period<K>() ? eo_table_bytes<K, PREC>()
                                : (PREC == PREC_FP32 ? f32_table_bytes<K>() : bf16_table_bytes<K>());
}
template <int K, int PREC>
__host__ __device__ constexpr int decide_mix_lds_bytes()
{
    return (PREC == PREC_BF16X3 ? 2 : 1) * mix_tab_bytes<K, PREC>() + mix_ytab_lds_bytes<K, PREC>() +
           mix_rv_bytes<K>();
}

template <int K, int PREC>
__global__ void __launch_bounds__(kMixBlock) k_decide_mix(KernelArgs a, const int *plist, int n_plist)
{
    extern __shared__ __attribute__((aligned(16))) char lds[];
    __shared__ DeferList deferred;
    deferred.begin();
    constexpr bool EO = mix_half_period<K>();
    constexpr int tab = mix_tab_bytes<K, PREC>();
    constexpr int phi_bytes = (PREC == PREC_BF16X3 ? 2 : 1) * tab;
    constexpr int yb = PREC == PREC_FP32 ? mix_ytab_f32_bytes<K>() : mix_ytab_bf16_bytes<K>();
    constexpr int ytab_bytes = mix_ytab_lds_bytes<K, PREC>();
    constexpr int rv_bytes = mix_rv_bytes<K>();
    static_assert(phi_bytes % 16 == 0 && ytab_bytes % 16 == 0 && rv_bytes % 16 == 0, "16-byte staging");
    if constexpr (EO) {
        stage_eo_tables<K, PREC, kMixBlock>(lds, a.phi_hi, a.phi_lo);
    } else {
        const uint4 *s0 = reinterpret_cast<const uint4 *>(a.phi_hi);
        uint4 *d = reinterpret_cast<uint4 *>(lds);
        for (int v = threadIdx.x; v < tab / 16; v += kMixBlock) d[v] = s0[v];
        if constexpr (PREC == PREC_BF16X3) {
            const uint4 *s1 = reinterpret_cast<const uint4 *>(a.phi_lo);
            for (int v = threadIdx.x; v < tab / 16; v += kMixBlock) d[tab / 16 + v] = s1[v];
        }
    }
    const char *lds_hi = lds;
    const char *lds_lo = lds + tab;
    const char *y_hi = lds + phi_bytes;
    const char *y_lo = lds + phi_bytes + yb;
    const float *rv = reinterpret_cast<const float *>(lds + phi_bytes + ytab_bytes);
    const PairCarry<6> carry{reinterpret_cast<float *>(lds + phi_bytes + ytab_bytes + rv_bytes) +
                             (threadIdx.x >> 6) * (PairCarry<6>::BYTES / 4)};
    const int lane = threadIdx.x & 63, half = lane >> 5, pl = lane & 31;
    const float Kf = (float)K;
    // the workgroups come to the points in turn: all waves share each queue
    const unsigned W = gridDim.x * (kMixBlock / kWave);
    const unsigned gwave = __builtin_amdgcn_readfirstlane(blockIdx.x * (kMixBlock / kWave) + (threadIdx.x >> 6));
    const float share = 1.0f / (2.0f * (float)W);
    for (int q = 0; q < n_plist; ++q) {
        const int p = __builtin_amdgcn_readfirstlane(plist[(blockIdx.x + q) % n_plist]);
        const DevPoint &P = a.pts[p];
        const DevMix &M = a.mix[p];
        DevCounters *C = a.cnt + p;
        __syncthreads();  // every wave is done with the previous point's tables
        {
            // y tables of the requested arithmetic, then the RV table
            const char *src = a.mix_tab + M.tab_off;
            const uint4 *sy = reinterpret_cast<const uint4 *>(
                src + (PREC == PREC_FP32 ? 2 * mix_ytab_bf16_bytes<K>() : 0));
            const uint4 *srv = reinterpret_cast<const uint4 *>(
                src + 2 * mix_ytab_bf16_bytes<K>() + mix_ytab_f32_bytes<K>());
            uint4 *dy = reinterpret_cast<uint4 *>(lds + phi_bytes);
            uint4 *drv = reinterpret_cast<uint4 *>(lds + phi_bytes + ytab_bytes);
            if constexpr (EO && PREC != PREC_FP32) {  // the parity layout of the split operands
                stage_parity_frags<K, kMixBlock>(dy, sy, 2);
                if constexpr (PREC == PREC_BF16X3) stage_parity_frags<K, kMixBlock>(dy + yb / 16, sy + yb / 16, 2);
            } else {
                for (int v = threadIdx.x; v < ytab_bytes / 16; v += kMixBlock) dy[v] = sy[v];
            }
            for (int v = threadIdx.x; v < rv_bytes / 16; v += kMixBlock) drv[v] = srv[v];
        }
        __syncthreads();
        PointTally tally;
        unsigned long long cur, end;
        static_range(P, p, gwave, W, cur, end);
        while (cur < end || claim_tiles<K>(P, C, lane, share, keeper_wave(p, gwave, W), cur, end)) {  // scalar branches
            const unsigned long long base = bcast_lane0(cur), left = bcast_lane0(end) - base;
            const int len = (int)(left < (unsigned long long)kClaimTiles ? left : (unsigned long long)kClaimTiles);
            cur = base + len;
            uint32_t my_word = 0u, my_def = 0u;
            const int len2 = (len + 1) & ~1;
        const unsigned long long stop = claim_stop(P, base, len);
#pragma unroll 1
            for (int c = 0; c < len2; ++c) {
                asm volatile("" ::: "memory");  // as in k_decide: no hoisting of the constants
                const unsigned long long tile = base + c;
                float x[K], r2, tk, qa;
                gen_x_mix_part<K, true>(P, M, rv, P.i0 + tile * kTile + pl, half, x, r2, tk, qa);
                carry.put(0, c & 1, lane, r2);
                carry.put(1, c & 1, lane, tk);
                qa = sum32(qa);
                if (a.dbg_xhat) {
                    const float inv = __builtin_amdgcn_rsqf(sum32(r2));
                    const unsigned long long local = tile * kTile + pl;
                    if (local < stop) {
#pragma unroll
                        for (int j = 0; j < K; ++j) a.dbg_xhat[local * (2 * K) + half * K + j] = x[j] * inv;
                    }
                }
                float sum = 0.0f, lmin = 0.0f;
                float s3l;
                f32x16 y0, y1;
                if constexpr (EO && PREC == PREC_FP32) {
                    s3l = cube_sum_eo_f32<K, 1>(x, lds_hi, lane);
                    bf16x8 bh[K / 8], bl[K / 8];
                    mix_y<K, PREC>(x, bh, bl, y_hi, y_lo, lane, y0, y1);
                } else if constexpr (EO && PREC == PREC_BF16X3) {
                    constexpr int S = eo_steps<K>();
                    bf16x8 eh[S], el[S], oh[S], ol[S];
                    split_eo<K, PREC>(x, eh, el, oh, ol);
                    // the shifts first: their sum is settled before the cube sum's accumulators
                    mix_y_eo<K, PREC>(x, eh, el, oh, ol, y_hi, y_lo, lane, y0, y1);
                    sum = mix_shift_sum(y0, y1, qa, Kf, lmin);
                    carry.put(3, c & 1, lane, sum);
                    carry.put(4, c & 1, lane, qa);
                    carry.put(5, c & 1, lane, lmin);
                    __builtin_amdgcn_sched_barrier(0);
                    s3l = cube_sum_eo_bf16<K, PREC, 1>(eh, el, oh, ol, lds_hi, lds_lo, lane);
                } else if constexpr (EO) {  // BF16: hi operands only
                    constexpr int S = eo_steps<K>();
                    bf16x8 eh[S], oh[S];
                    split_eo_hi<K>(x, eh, oh);
                    s3l = cube_sum_eo_bf16<K, PREC, 1>(eh, nullptr, oh, nullptr, lds_hi, lds_lo, lane);
                    mix_y_eo<K, PREC>(x, eh, nullptr, oh, nullptr, y_hi, y_lo, lane, y0, y1);
                } else {
                    bf16x8 bh[K / 8], bl[K / 8];
                    if constexpr (PREC != PREC_FP32) split_bf16<K, PREC>(x, bh, bl);
                    s3l = cube_sum_ops<K, PREC>(x, bh, bl, lds_hi, lds_lo, lane);
                    mix_y<K, PREC>(x, bh, bl, y_hi, y_lo, lane, y0, y1);
                }
                if constexpr (!(EO && PREC == PREC_BF16X3)) sum = mix_shift_sum(y0, y1, qa, Kf, lmin);
                carry.put(2, c & 1, lane, s3l);
                if constexpr (!(EO && PREC == PREC_BF16X3)) {
                    carry.put(3, c & 1, lane, sum);
                    carry.put(4, c & 1, lane, qa);
                    carry.put(5, c & 1, lane, lmin);
                }
                if ((c & 1) == 0) continue;
                // settle both tiles at once, a proposal per lane (k_decide)
                wave_lds_sync();
                asm volatile("" ::: "memory");
                const float inv = __builtin_amdgcn_rsqf(carry.sum(0, half, pl));
                const float t = carry.sum(1, half, pl) * (inv * inv);
                const float s3 = carry.sum(2, half, pl) * (inv * inv * inv);
                const float lq = mix_log_q_f32(P, M, carry.sum(3, half, pl), carry.first(5, half, pl),
                                               carry.first(4, half, pl), inv * inv, t, Kf);
                wave_lds_sync();
                const float lf = __builtin_fmaf(P.neg_bp_K2, t, P.c3coef * s3);
                const float la = (lf - lq) - P.log_M;
                const unsigned long long local = (tile - 1) * kTile + lane;
                const bool valid = local < stop;
                const uint32_t w_acc = acceptance_word<K>(P, P.i0 + local);
                bool accept, defer;
                verdict(P, la, w_acc, valid, accept, defer);
                const unsigned long long bacc = __ballot(accept);
                const unsigned long long bdef = __ballot(defer);
                if ((lane | 1) == c) my_word = (uint32_t)((lane & 1) ? bacc >> 32 : bacc);
                if (bdef) {
                    if ((lane | 1) == c) my_def = (uint32_t)((lane & 1) ? bdef >> 32 : bdef);
                }
                if (valid) {
                    tally.n_viol += (la > 0.0f && !defer) ? 1u : 0u;  // window proposals: k_fixup_mix
                    tally.max_la = fmaxf(tally.max_la, la);
                    if (a.dbg_t) {
                        a.dbg_t[local] = t;
                        a.dbg_s3[local] = s3;
                        a.dbg_log_a[local] = la;
                        a.dbg_log_u[local] = log_u_word(w_acc);
                    }
                }
            }
            if (lane < len) a.bitmap[P.bm_off + base + lane] = my_word;
            deferred.push(a, C, p, P.i0 + base * kTile, my_def, lane);
            count_accepted(P, C, my_word, len, lane);
        }
        tally.report(C, lane);
    }
    deferred.flush(a);
}

// ---------------------------------------------------------------------------
// k_fixup: FP64 evaluation of listed proposals, as the paper states it:
// normals from the same words, X = Sigma^{1/2} z, X^ = X/|X|, H2 by Parseval,
// H3 by the double sum, log f/(M g) = -beta H + K log(1 + alpha beta' t/K^3) - log M.
//
// K/2 lanes take one proposal (128/K proposals per wave): lane l draws Philox
// block l, i.e. coordinates 4l .. 4l+3, and after the projection sums the
// triads of two third modes, n = l + 2 and n = K - l, which together have K
// terms for every l; the inner sum's symmetry k <-> n - k halves them.  A list
// holds some 1e-4 to 1e-2 of a call's proposals, too few to fill the chip with
// one thread each, and one thread's 2K coordinates lived in scratch memory: the
// kernel took 0.6 ms for 83 thousand proposals at K = 16, 2.0 ms for 700 at
// K = 128; split over lanes 0.03 ms and 0.02 ms.
// ---------------------------------------------------------------------------
constexpr double kRoundLogA = 0x1p-48;  // 32 roundings of each term: five operations a term, a log1p, log M's own
template <int K>
__global__ void __launch_bounds__(kBlock) k_fixup(KernelArgs a, int plan)
{
    // the last workgroup lays out the segments (they depend on the decided range only)
    if (plan && blockIdx.x == gridDim.x - 1) plan_segments<kBlock>(a);
    constexpr int LP = K / 2, PER = kWave / LP;  // lanes per proposal, proposals per wave
    static_assert(LP * PER == kWave, "K/2 lanes per proposal");
    __shared__ double xs[kBlock / kWave][PER * 2 * K];
    const int lane = threadIdx.x & 63, l = lane % LP, grp = lane / LP;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    double *x = xs[wv] + grp * 2 * K;
    auto group_sum = [](double v) {
#pragma unroll
        for (int o = LP / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
        return v;
    };
    const unsigned long long cnt = *a.defer_count;
    const unsigned long long n = cnt < a.defer_cap ? cnt : a.defer_cap;
    const unsigned long long nw = (unsigned long long)gridDim.x * (kBlock / kWave);
    for (unsigned long long e0 = (unsigned long long)PER * ((unsigned long long)blockIdx.x * (kBlock / kWave) + wv);
         e0 < n; e0 += (unsigned long long)PER * nw) {
        // groups past the end repeat the first entry; their result is not used
        const bool item = e0 + grp < n;
        const unsigned long long v = a.defer_list[item ? e0 + grp : e0];
        const int p = (int)(v >> 40);
        const uint64_t i = v & ((1ull << 40) - 1ull);
        const DevPoint &P = a.pts[p];
        const bool mine = item && P.K == K;  // a list may hold points of several K, each with its launch
        if (__ballot(mine) == 0ull) continue;
        const uint32_t c0 = (uint32_t)i, c1 = (uint32_t)(i >> 32);
        double X[4];
        {
            const uint4 w = philox4x32_10(c0, c1, P.point_id, (uint32_t)l, P.key0, P.key1);
            const uint32_t ws[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
            for (int q = 0; q < 4; q += 2) {
                const double u1 = ((double)ws[q] + 0.5) * 0x1p-32;
                const double u2 = ((double)ws[q + 1] + 0.5) * 0x1p-32;
                const double r = sqrt(-2.0 * log(u1));
                double sn, cs;
                sincospi(2.0 * u2, &sn, &cs);
                X[q] = r * cs;
                X[q + 1] = r * sn;
            }
        }
        const uint32_t w_acc = philox4x32_10(c0, c1, P.point_id, (uint32_t)(K / 2), P.key0, P.key1).x;
        const int k0 = (4 * l) % K;  // this lane's modes are k0 + 1 .. k0 + 4 of one block
        double r2 = 0.0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            X[q] *= P.sig64[k0 + q];
            r2 += X[q] * X[q];
        }
        const double r = sqrt(group_sum(r2));
        double tk = 0.0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            X[q] /= r;
            x[4 * l + q] = X[q];
            tk += (double)((k0 + q + 1) * (k0 + q + 1)) * X[q] * X[q];
        }
        const double t = group_sum(tk);
        // the wave's copies of x^ are written and read by its own lanes only
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
        // sum over n of x_n Re + x_{K+n} Im of the inner sums over k + (n - k) = n
        double tri = 0.0;
        {
            const int n1 = l + 2, n2 = K - l;
            const int h1 = n1 <= n2 ? n1 / 2 : 0, h2 = n1 < n2 ? n2 / 2 : 0;  // terms k <= n/2
            const double a1 = x[n1 - 1], b1 = x[K + n1 - 1], a2 = x[n2 - 1], b2 = x[K + n2 - 1];
            for (int it = 0; it < h1 + h2; ++it) {
                const bool first = it < h1;
                const int nn = first ? n1 : n2, k = (first ? it : it - h1) + 1, m = nn - k;
                const double an = first ? a1 : a2, bn = first ? b1 : b2;
                const double ck = x[k - 1], sk = x[K + k - 1], cm = x[m - 1], sm = x[K + m - 1];
                const double term = an * (ck * cm - sk * sm) + bn * (ck * sm + sk * cm);
                tri += k == m ? term : 2.0 * term;
            }
        }
        const double pi = 3.14159265358979323846;
        const double s = sqrt(P.E0 / (2.0 * pi));
        const double H3 = 2.0 * pi * (s * s * s) * group_sum(tri);
        const double bh = P.beta_p / (P.E0 * (double)K * K);
        double lr = -(bh * (P.E0 * t - P.c32 * H3)), lg = 0.0;
        if (P.proposal == PROP_SIGMA) {
            lg = K * log1p(P.alpha_star * P.beta_p * t / ((double)K * K * K));
            lr += lg;
        }
        const double la = lr - P.log_M64, lu = log(((double)w_acc + 0.5) * 0x1p-32);
        // the rounding of la's terms where it is near 0: with an exact M (C3/C2 = 0) f/(M g)
        // comes as near to 1 as that, and there t's own error does not count (its maximum)
        const double eps = kRoundLogA * (bh * (P.E0 * t + fabs(P.c32 * H3)) + lg + fabs(P.log_M64));
        if (mine && l == 0) {
            if (lu < la) {
                const uint64_t local = i - P.i0;
                atomicOr(&a.bitmap[P.bm_off + local / 32], 1u << (local % 32));
            }
            if (la > eps) {  // f/(M g) > 1 (eq. M_sup broken): counted here for window proposals
                atomicAdd(&a.cnt[p].shard[0].violations, 1ull);
                atomicMax(&a.cnt[p].shard[0].max_log_a_key, float_key((float)la));
            }
        }
        // the next proposals overwrite this wave's copies of x^
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
}

// ---------------------------------------------------------------------------
// k_fixup_mix: FP64 re-decision of listed proposals of the mixture sampler.
// Each half-wave takes one proposal (two per wave), lane l of the half:
//   * the Box-Muller pair l (coordinates 2l, 2l+1) of the draw of gen_x_mix
//     in FP64, the component from the same word, in integers;
//   * mode n = l + 2 of the double sum over triads of H3;
//   * shift j = l of q_net: x^T L0^-1 x of w = R_j^T x^ as e^T A e + |g|^2,
//     g = G^-1 V^T A w, e = w - V g (no cancellation), over all K modes;
// then a half-wave log-sum-exp over the shifts.
// log a = log f - log q_mix - log M.
// ---------------------------------------------------------------------------
__device__ __forceinline__ double half_sum_f64(double v)
{
#pragma unroll
    for (int o = 16; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}
__device__ __forceinline__ double half_max_f64(double v)
{
#pragma unroll
    for (int o = 16; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
    return v;
}
template <int K>
__global__ void __launch_bounds__(kBlock) k_fixup_mix(KernelArgs a, int plan)
{
    // the last workgroup lays out the segments (they depend on the decided range only)
    if (plan && blockIdx.x == gridDim.x - 1) plan_segments<kBlock>(a);
    static_assert(K <= 32 && kMixS == 32, "one lane per Box-Muller pair, triad mode and shift");
    __shared__ double xs[kBlock / kWave][2][2 * K];
    const int lane = threadIdx.x & 63, h = lane >> 5, l = lane & 31;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    double *x = xs[wv][h];
    const double pi = 3.14159265358979323846;
    const unsigned long long cnt = *a.defer_count;
    const unsigned long long n = cnt < a.defer_cap ? cnt : a.defer_cap;
    const unsigned long long nw = (unsigned long long)gridDim.x * (kBlock / kWave);
    for (unsigned long long e0 = 2ull * ((unsigned long long)blockIdx.x * (kBlock / kWave) + wv); e0 < n;
         e0 += 2ull * nw) {
        // a second half past the end repeats the first half's proposal; its
        // result is not used
        const bool item = e0 + h < n;
        const unsigned long long v = a.defer_list[item ? e0 + h : e0];
        const int p = (int)(v >> 40);
        const uint64_t i = v & ((1ull << 40) - 1ull);
        const DevPoint &P = a.pts[p];
        const DevMix &M = a.mix[p];
        const uint32_t c0 = (uint32_t)i, c1 = (uint32_t)(i >> 32);
        const uint4 wl = philox4x32_10(c0, c1, P.point_id, (uint32_t)(K / 2), P.key0, P.key1);
        const int comp = wl.y < M.E ? -1 : (int)((wl.y - M.E) / M.B);
        // eta pair of the component (every lane; used when comp >= 0)
        double e0v = 0.0, e1v = 0.0;
        if (comp >= 0) {
            const double r = sqrt(-2.0 * log(((double)wl.z + 0.5) * 0x1p-32));
            const double th = 2.0 * pi * (((double)wl.w + 0.5) * 0x1p-32);
            e0v = r * cos(th);
            e1v = r * sin(th);
        }
        // coordinate m from its normal z
        auto coord = [&](int m, double z) {
            const int k = m % K + 1;
            if (comp < 0) return P.sig64[k - 1] * z;
            const int mi = (k * comp) & (kMixS - 1);
            const double cs = M.cs64[mi], sn = M.sn64[mi];
            const double *vc = M.V64[k - 1], *vs = M.V64[K + k - 1];
            const bool sinb = m >= K;
            const double r0 = sinb ? vs[0] * cs - vc[0] * sn : vc[0] * cs + vs[0] * sn;
            const double r1 = sinb ? vs[1] * cs - vc[1] * sn : vc[1] * cs + vs[1] * sn;
            return M.sqd64[k - 1] * z + r0 * e0v + r1 * e1v;
        };
        double X0 = 0.0, X1 = 0.0;
        if (l < K) {
            const uint4 w = philox4x32_10(c0, c1, P.point_id, (uint32_t)(l / 2), P.key0, P.key1);
            const uint32_t w1 = (l & 1) ? w.z : w.x, w2 = (l & 1) ? w.w : w.y;
            const double r = sqrt(-2.0 * log(((double)w1 + 0.5) * 0x1p-32));
            const double th = 2.0 * pi * (((double)w2 + 0.5) * 0x1p-32);
            X0 = coord(2 * l, r * cos(th));
            X1 = coord(2 * l + 1, r * sin(th));
        }
        const double inv_r = 1.0 / sqrt(half_sum_f64(X0 * X0 + X1 * X1));
        const double x0 = X0 * inv_r, x1 = X1 * inv_r;
        if (l < K) {
            x[2 * l] = x0;
            x[2 * l + 1] = x1;
        }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
        double tk = 0.0;
        if (l < K) {
            const double k0 = (2 * l) % K + 1, k1 = (2 * l + 1) % K + 1;
            tk = k0 * k0 * x0 * x0 + k1 * k1 * x1 * x1;
        }
        const double t = half_sum_f64(tk);
        // H3 by the double sum: lane l takes n = l + 2
        double tri = 0.0;
        {
            const int nn = l + 2;
            if (nn <= K) {
                const double s = sqrt(P.E0 / (2.0 * pi));
                double in_re = 0.0, in_im = 0.0;
                for (int kk = 1; kk < nn; ++kk) {
                    const double pr = s * x[kk - 1], pi_ = -s * x[K + kk - 1];
                    const double qr = s * x[nn - kk - 1], qi = -s * x[K + nn - kk - 1];
                    in_re += pr * qr - pi_ * qi;
                    in_im += pr * qi + pi_ * qr;
                }
                tri = (s * x[nn - 1]) * in_re + (-s * x[K + nn - 1]) * in_im;
            }
        }
        const double H3 = 2.0 * pi * half_sum_f64(tri);
        const double lf = -(P.beta_p / (P.E0 * (double)K * K) * (P.E0 * t - P.c32 * H3));
        // q_net: shift j = l
        double y0 = 0.0, y1 = 0.0;
#pragma unroll 4
        for (int k = 1; k <= K; ++k) {
            const int mi = (k * l) & (kMixS - 1);
            const double cs = M.cs64[mi], sn = M.sn64[mi];
            const double xc = x[k - 1], xsn = x[K + k - 1];
            const double wc = xc * cs - xsn * sn, ws = xsn * cs + xc * sn;
            const double ak = M.a64[k - 1];
            y0 += ak * (M.V64[k - 1][0] * wc + M.V64[K + k - 1][0] * ws);
            y1 += ak * (M.V64[k - 1][1] * wc + M.V64[K + k - 1][1] * ws);
        }
        const double g0 = M.gi64[0][0] * y0 + M.gi64[0][1] * y1;
        const double g1 = M.gi64[1][0] * y0 + M.gi64[1][1] * y1;
        double qf = g0 * g0 + g1 * g1;
#pragma unroll 4
        for (int k = 1; k <= K; ++k) {
            const int mi = (k * l) & (kMixS - 1);
            const double cs = M.cs64[mi], sn = M.sn64[mi];
            const double xc = x[k - 1], xsn = x[K + k - 1];
            const double wc = xc * cs - xsn * sn, ws = xsn * cs + xc * sn;
            const double ec = wc - (M.V64[k - 1][0] * g0 + M.V64[k - 1][1] * g1);
            const double es = ws - (M.V64[K + k - 1][0] * g0 + M.V64[K + k - 1][1] * g1);
            qf += M.a64[k - 1] * (ec * ec + es * es);
        }
        const double lj = -K * log(qf);
        const double mx = half_max_f64(lj);
        const double se = half_sum_f64(exp(lj - mx));
        const double lnet = -0.5 * M.logdetL0 + mx + log(se) - log((double)kMixS);
        const double lg = M.lng - K * log1p(P.alpha_star * P.beta_p * t / ((double)K * K * K));
        const double A = M.log_eps + lg, B = M.log_1m_eps + lnet;
        const double hi = A > B ? A : B;
        const double lq = hi + log(exp(A - hi) + exp(B - hi));
        const double log_u = log(((double)wl.x + 0.5) * 0x1p-32);
        const double log_a = lf - lq - P.log_M64;
        // updates of each half in turn, under a wave-uniform condition at a
        // wave-uniform address (lane 0 of the wave carries the value)
        const bool acc = item && log_u < log_a;
        const bool viol = item && log_a > 0.0;  // f/(M q_mix) > 1, counted here for window proposals
        const unsigned long long bm_word = P.bm_off + (i - P.i0) / 32;
        const uint32_t bit = 1u << ((i - P.i0) % 32);
#pragma unroll
        for (int hh = 0; hh < 2; ++hh) {
            if (__builtin_amdgcn_readlane((int)acc, 32 * hh) != 0) {
                const unsigned long long wrd = read_lane_u64(bm_word, 32 * hh);
                const uint32_t b = __builtin_amdgcn_readlane(bit, 32 * hh);
                atomicOr(&a.bitmap[wrd], lane == 0 ? b : 0u);
            }
            if (__builtin_amdgcn_readlane((int)viol, 32 * hh) != 0) {
                const int pp = __builtin_amdgcn_readlane(p, 32 * hh);
                const unsigned int key = __builtin_amdgcn_readlane(float_key((float)log_a), 32 * hh);
                atomicAdd(&a.cnt[pp].shard[0].violations, lane == 0 ? 1ull : 0ull);
                atomicMax(&a.cnt[pp].shard[0].max_log_a_key, lane == 0 ? key : 0u);
            }
        }
        // the next proposals overwrite this wave's copies of x^
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
}

// ---------------------------------------------------------------------------
// Segments: accept counts (a wave per segment) and their prefix.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(kBlock) k_seg_count(KernelArgs a)
{
    const int lane = threadIdx.x & 63;
    const unsigned long long total = cut_first(a.seg, a.n_points);
    const unsigned long long waves = (unsigned long long)gridDim.x * (kBlock / kWave);
    for (unsigned long long gs = __builtin_amdgcn_readfirstlane(blockIdx.x * (kBlock / kWave) + (threadIdx.x >> 6));
         gs < total; gs += waves) {
        const int p = __builtin_amdgcn_readfirstlane(point_of_cut(a.seg, a.n_points, gs, lane));
        const DevPoint &P = a.pts[p];
        const unsigned long long nw = tiles_taken(P, a.cnt[p].next_tile);
        const unsigned long long S = 1ull << cut_shift(a.seg, p), w0 = (gs - cut_first(a.seg, p)) * S;
        const unsigned long long w1 = w0 + S < nw ? w0 + S : nw;
        unsigned int c = 0;
#pragma unroll 4
        for (unsigned long long w = w0 + lane; w < w1; w += kWave) c += __popc(a.bitmap[P.bm_off + w]);
        c = wave_sum_u32(c);
        if (lane == 0) a.seg_cnt[gs] = c;
    }
}

// One workgroup: exclusive prefix of the segments' counts (each thread a contiguous
// run of them), the points' totals and their runs of ranks.
__global__ void __launch_bounds__(1024) k_seg_scan(KernelArgs a)
{
    __shared__ unsigned long long wsum[16];
    const int tid = threadIdx.x, seg_shift = cut_shift(a.seg, 0);
    const unsigned long long n = cut_first(a.seg, a.n_points);
    // of the first point, beside the scan's loads: all there is for a point alone
    const int K0 = a.pts[0].K;
    const unsigned long long words0 = tiles_taken(a.pts[0], a.cnt[0].next_tile), last0 = a.pts[0].n, target0 = a.pts[0].target;
    const unsigned long long per = (n + 1023) / 1024, b = per * tid < n ? per * tid : n, e = b + per < n ? b + per : n;
    unsigned long long own = 0;
#pragma unroll 8
    for (unsigned long long s = b; s < e; ++s) own += a.seg_cnt[s];
    unsigned long long all;
    unsigned long long run = block_prefix<1024>(own, wsum, all);
#pragma unroll 8
    for (unsigned long long s = b; s < e; ++s) {
        a.seg_base[s] = run;
        run += a.seg_cnt[s];
    }
    if (tid == 0) a.seg_base[n] = all;
    // point p of the segments [s0, s1), the accepted before each: its runs
    auto point = [&](int p, unsigned long long words, unsigned long long last, unsigned long long target, int K,
                     unsigned long long s0, unsigned long long s1, unsigned long long base, unsigned long long upto,
                     int &sh) {
        const unsigned long long done = words * kTile, accepted = upto - base;
        const unsigned long long samples = accepted < target ? accepted : target;
        a.ranks[p] = PointRanks{samples, s0, s1 - s0, base, words, seg_shift, 0};
        a.res[p].n_accepted = accepted;
        a.res[p].n_processed = done < last ? done : last;
        sh = run_shift(K, samples);
        return runs_of(K, samples);
    };
    if (a.n_points == 1) {
        if (tid != 0) return;
        int sh;
        a.runs->at[1] = point(0, words0, last0, target0, K0, 0ull, n, 0ull, all, sh);
        a.runs->at[0] = (unsigned long long)sh << kCutShiftBit;
        return;
    }
    __syncthreads();  // the points read what other threads wrote
    place_cuts<1024>(a.runs, a.n_points, [&](int p, int &sh) {
        const unsigned long long s0 = cut_first(a.seg, p), s1 = cut_first(a.seg, p + 1);
        const DevPoint &P = a.pts[p];
        return point(p, tiles_taken(P, a.cnt[p].next_tile), P.n, P.target, P.K, s0, s1, a.seg_base[s0], a.seg_base[s1], sh);
    });
}

// ---------------------------------------------------------------------------
// k_materialize: one wave per run of ranks; no work past the accepted-sample
// target (dense words beyond it cost a map of 500 samples per cell 26 ms of 37).
// ---------------------------------------------------------------------------
using Ranks = RankReader<kWave, kTile>;

template <int K>
__host__ __device__ constexpr int materialize_tab_bytes()
{
    // the FP32 table; for K >= 16 its first half (the half-period form)
    return K >= 16 ? eo_table_bytes<K, PREC_FP32>() : f32_table_bytes<K>();
}
template <int K>
__host__ __device__ constexpr int materialize_lds_bytes()
{
    return materialize_tab_bytes<K>() + (kBlock / kWave) * (Ranks::N * 2 + kNBins * 4);
}

template <int K, int PROP>
__global__ void __launch_bounds__(kBlock) k_materialize(KernelArgs a, float *out_xhat, unsigned long long *out_index)
{
    extern __shared__ __attribute__((aligned(16))) char lds[];
    constexpr int tab = materialize_tab_bytes<K>();
    const unsigned long long total = cut_first(a.runs, a.n_points);
    if ((unsigned long long)blockIdx.x * (kBlock / kWave) >= total) return;
    {
        const uint4 *s0 = reinterpret_cast<const uint4 *>(a.phi_hi);
        uint4 *d = reinterpret_cast<uint4 *>(lds);
        for (int v = threadIdx.x; v < tab / 16; v += kBlock) d[v] = s0[v];
    }
    const int lane = threadIdx.x & 63, half = lane >> 5, pl = lane & 31;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint16_t *mylist = reinterpret_cast<uint16_t *>(lds + tab) + wv * Ranks::N;
    WaveHist hist;
    hist.bins = reinterpret_cast<unsigned int *>(lds + tab + (kBlock / kWave) * Ranks::N * 2) + wv * kNBins;
    __syncthreads();
    const unsigned long long waves = (unsigned long long)gridDim.x * (kBlock / kWave);
    for (unsigned long long run = (unsigned long long)blockIdx.x * (kBlock / kWave) + wv; run < total; run += waves) {
        const int p = __builtin_amdgcn_readfirstlane(point_of_cut(a.runs, a.n_points, run, lane));
        const DevPoint &P = a.pts[p];
        if (P.K != K || P.proposal != PROP) continue;
        hist.enter(a, p, lane);
        const PointRanks &R = a.ranks[p];
        const int sh = cut_shift(a.runs, p);
        const unsigned long long first = (run - cut_first(a.runs, p)) << sh, n = R.samples;
        Ranks ranks(a, R, P.bm_off, mylist, first, n - first < (1ull << sh) ? n : first + (1ull << sh), lane);
        GridSums sums;
        unsigned int n_max4 = 0;
        unsigned long long peak_idx = ~0ull;
        unsigned int peak_key = 0u;
        while (const int upto = ranks.next(lane)) {
            for (int c0 = 0; c0 < upto; c0 += kTile) {
                const bool valid = c0 + pl < upto;
                const uint64_t i = P.i0 + (valid ? ranks.local(c0 + pl) : 0ull);
                const unsigned long long r = ranks.rank + c0 + pl;
                float x[K];
                float t;
                if constexpr (PROP == PROP_MIXTURE) {
                    const DevMix &M = a.mix[p];
                    const float *rvg = reinterpret_cast<const float *>(
                        a.mix_tab + M.tab_off + 2 * mix_ytab_bf16_bytes<K>() + mix_ytab_f32_bytes<K>());
                    gen_xhat_mix<K>(P, M, rvg, i, half, x, t);
                } else {
                    gen_xhat<K, PROP>(P, i, half, x, t);
                }
                if (valid && r < P.capacity) {
                    if (out_xhat) {
                        float *row = out_xhat + (P.out_off + r) * P.row_stride + half * K;
#pragma unroll
                        for (int j = 0; j < K; ++j) row[j] = x[j];
                    }
                    if (out_index && half == 0) out_index[P.out_off + r] = i;
                }
                if (valid && half == 0 && r + 1 == P.target) a.cnt[p].last_index = i;
                // statistics on the grid: u = sqrt(2 E0/pi) u~, u~ from FP32 products
                // (K >= 16: the half-period form, u~ = E + O and E - O on the two halves)
                const float4 *ftab = reinterpret_cast<const float4 *>(lds);
                if (__any(!valid)) {  // no sample, no contribution: u~ = 0
#pragma unroll
                    for (int j = 0; j < K; ++j) x[j] = valid ? x[j] : 0.0f;
                }
                sums.umax = -INFINITY;
                if constexpr (K >= 16) {
#pragma unroll
                    for (int tp = 0; tp < K / 16; ++tp) {
                        f32x16 ce = {}, co = {};
#pragma unroll
                        for (int q = 0; q < K / 4; ++q) {
                            // entries 0..3: modes 4q+1 (odd), 4q+2 (even), 4q+3 (odd), 4q+4 (even)
                            const float4 av = ftab[(tp * (K / 4) + q) * kWave + lane];
                            co = __builtin_amdgcn_mfma_f32_32x32x2f32(av.x, x[4 * q + 0], co, 0, 0, 0);
                            ce = __builtin_amdgcn_mfma_f32_32x32x2f32(av.y, x[4 * q + 1], ce, 0, 0, 0);
                            co = __builtin_amdgcn_mfma_f32_32x32x2f32(av.z, x[4 * q + 2], co, 0, 0, 0);
                            ce = __builtin_amdgcn_mfma_f32_32x32x2f32(av.w, x[4 * q + 3], ce, 0, 0, 0);
                        }
                        float u[32];
#pragma unroll
                        for (int v = 0; v < 16; ++v) {
                            u[2 * v] = ce[v] + co[v];
                            u[2 * v + 1] = ce[v] - co[v];
                        }
                        sums.add(u);
                    }
                } else {
#pragma unroll
                    for (int tt = 0; tt < K / 8; ++tt) {
                        f32x16 acc = {};
#pragma unroll
                        for (int q = 0; q < K / 4; ++q) {
                            const float4 av = ftab[(tt * (K / 4) + q) * kWave + lane];
                            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(av.x, x[4 * q + 0], acc, 0, 0, 0);
                            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(av.y, x[4 * q + 1], acc, 0, 0, 0);
                            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(av.z, x[4 * q + 2], acc, 0, 0, 0);
                            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(av.w, x[4 * q + 3], acc, 0, 0, 0);
                        }
                        float u[16];
#pragma unroll
                        for (int v = 0; v < 16; ++v) u[v] = acc[v];
                        sums.add(u);
                    }
                }
                // the proposal's grid values are split over lanes l and l + 32
                const float umax = fmaxf(sums.umax, __shfl_xor(sums.umax, 32, 64));
                if (valid && half == 0) {
                    n_max4 += umax > kFourSigmaT ? 1u : 0u;
                    peak_merge(peak_key, peak_idx, float_key(umax), i);
                }
                if (valid && half == 0) {
                    // u(0) = sqrt(2 E0/pi) sum_k x^_k; bin of u(0)/u_max = sum_k x^_k / sqrt(K)
                    double s0 = 0.0;
#pragma unroll
                    for (int j = 0; j < K; ++j) s0 += (double)x[j];
                    double posb = (s0 / sqrt((double)K) + 1.0) * (0.5 * kNBins);
                    int bin = (int)floor(posb);
                    bin = bin < 0 ? 0 : (bin > kNBins - 1 ? kNBins - 1 : bin);
                    atomicAdd(&hist.bins[bin], 1u);
                }
            }
            ranks.done(upto, lane);
        }
        const double amp2 = P.amp * P.amp;
        const double S1 = P.amp * wave_sum_f64(sums.S1), S2 = amp2 * wave_sum_f64(sums.S2);
        const double S3 = amp2 * P.amp * wave_sum_f64(sums.S3), S4 = amp2 * amp2 * wave_sum_f64(sums.S4);
        n_max4 = wave_sum_u32(n_max4);
        wave_peak(peak_key, peak_idx);
        if (lane == 0)
            a.run_stats[run] = RunStats{S1, S2, S3, S4, peak_idx, peak_key, sums.n_ex, sums.n_ex4, n_max4};
    }
    hist.flush(a, lane);
}

// Per point (one workgroup): the runs' partials summed in a fixed order -- each
// thread takes every 1024th run in order, then a fixed pairwise tree over the
// threads -- so that the result depends on the accepted samples alone.
constexpr int kFinBlock = 1024;
__global__ void __launch_bounds__(kFinBlock) k_finalize(KernelArgs a)
{
    __shared__ double sS[4][kFinBlock / kWave];
    __shared__ unsigned long long sE[3][kFinBlock / kWave], sPI[kFinBlock / kWave];
    __shared__ unsigned int sPK[kFinBlock / kWave];
    if (a.d_active && *a.d_active == 0ull) return;
    const int p = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const DevPoint &P = a.pts[p];
    const unsigned long long r0 = cut_first(a.runs, p), r1 = cut_first(a.runs, p + 1), n = a.ranks[p].samples;
    double S[4] = {0.0, 0.0, 0.0, 0.0};
    unsigned long long E[3] = {0, 0, 0}, pi = ~0ull;  // above 2 sigma, 4 sigma, samples above 4 sigma
    unsigned int pk = 0u;
    // the next record's loads are issued beside this one's sums
#pragma unroll 2
    for (unsigned long long r = r0 + tid; r < r1; r += kFinBlock) {
        const RunStats st = a.run_stats[r];
        S[0] += st.S1;
        S[1] += st.S2;
        S[2] += st.S3;
        S[3] += st.S4;
        E[0] += st.n_exceed;
        E[1] += st.n_exceed4;
        E[2] += st.n_max4;
        peak_merge(pk, pi, st.peak_key, st.peak_index);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) S[q] = wave_sum_f64(S[q]);
#pragma unroll
    for (int q = 0; q < 3; ++q)
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) E[q] += __shfl_xor(E[q], o, 64);
    wave_peak(pk, pi);
    if (lane == 0) {
        for (int q = 0; q < 4; ++q) sS[q][wv] = S[q];
        for (int q = 0; q < 3; ++q) sE[q][wv] = E[q];
        sPK[wv] = pk;
        sPI[wv] = pi;
    }
    __syncthreads();
    PointResult &R = a.res[p];
    if (tid < kNBins) {
        unsigned long long h = 0;
        for (int s = 0; s < kShards; ++s) h += a.hist[((size_t)p * kShards + s) * kNBins + tid];
        R.hist[tid] = h;
    }
    if (wv != 0) return;
    // the waves' sums, a wave's by a lane (a loop of one thread over them was
    // unrolled into 138 spilled registers)
    const bool mine = lane < kFinBlock / kWave;
#pragma unroll
    for (int q = 0; q < 4; ++q) S[q] = wave_sum_f64(mine ? sS[q][lane] : 0.0);
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        E[q] = mine ? sE[q][lane] : 0ull;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) E[q] += __shfl_xor(E[q], o, 64);
    }
    pk = mine ? sPK[lane] : 0u;
    pi = mine ? sPI[lane] : ~0ull;
    wave_peak(pk, pi);
    if (lane == 0) {
        R.S1 = S[0];
        R.S2 = S[1];
        R.S3 = S[2];
        R.S4 = S[3];
        R.n_exceed = E[0];
        R.n_exceed4 = E[1];
        R.n_max4 = E[2];
        R.peak_key = pk;
        R.peak_index = pi;
        R.n_samples = n;
        R.n_written = n < P.capacity ? n : P.capacity;
    }
}

// ---------------------------------------------------------------------------
// k_window_advance: after one window of a sweep, one workgroup:
//   per point: fold the window's statistics into the running totals, count
//   the accepted samples (the window's target is what was still missing) and
//   mark the point done when its target is met or its index range used up
//   (a done point gets no tiles);
//   then, in point order: the next window of every active point -- its first
//   index, size, remaining target and capacity, output offset, and its place
//   in the window's accept bitmap.  Adaptive windows take the proposals the
//   point still needs at its measured acceptance, times 1.25 (four times the
//   proposals so far while it has accepted none), shared out of the bitmap pool
//   in proportion when they do not fit; otherwise every window has the first
//   window's size.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(1024) k_window_advance(DevPoint *pts, const DevCounters *cnt,
                                                         const PointResult *res, SweepState *sw, int n_points,
                                                         SweepGlobal *G, const unsigned long long *defer_count)
{
    __shared__ double need[1024];
    __shared__ int any_active;
    if (threadIdx.x == 0) any_active = 0;
    __syncthreads();
    for (int p = threadIdx.x; p < n_points; p += blockDim.x) {
        SweepState &S = sw[p];
        DevPoint &P = pts[p];
        if (S.done) continue;
        any_active = 1;
        const PointResult &r = res[p];
        const DevCounters &c = cnt[p];
        S.total.S1 += r.S1;
        S.total.S2 += r.S2;
        S.total.S3 += r.S3;
        S.total.S4 += r.S4;
        S.total.n_exceed += r.n_exceed;
        S.total.n_exceed4 += r.n_exceed4;
        S.total.n_max4 += r.n_max4;
        // windows come in increasing index: a later one replaces the peak only when larger
        if (r.peak_key > S.total.peak_key) {
            S.total.peak_key = r.peak_key;
            S.total.peak_index = r.peak_index;
        }
        for (int b = 0; b < kNBins; ++b) S.total.hist[b] += r.hist[b];
        S.accepted += r.n_samples;
        S.written += r.n_written;
        const CounterShard ct = shard_totals(c);
        S.n_fixups += ct.deferred;
        S.n_violations += ct.violations;
        if (ct.max_log_a_key > S.max_log_a_key) S.max_log_a_key = ct.max_log_a_key;
        if (S.accepted >= S.target) {
            S.n_proposed = c.last_index - S.i_start + 1;
            S.done = 1;
        } else {
            S.n_proposed += P.n;
            if (P.i0 + P.n >= S.i_end) S.done = 1;
        }
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    if (any_active) G->windows += 1;
    if (*defer_count > G->defer_cap) G->overflow = 1;
    // sizes of the next windows, in point order
    double sum_need = 0.0;
    for (int p = 0; p < n_points; ++p) {
        const SweepState &S = sw[p];
        const DevPoint &P = pts[p];
        if (S.done) continue;
        const double next_i0 = (double)(P.i0 + P.n), left = (double)S.i_end - next_i0;
        double w = (double)S.window;
        if (G->adaptive) {
            const double used = (double)(P.i0 + P.n - S.i_start);
            const double missing = (double)(S.target - S.accepted);
            w = S.accepted > 0 ? 1.25 * missing * used / (double)S.accepted : 4.0 * used;
            w = w < (double)S.window ? (double)S.window : w;
        }
        w = w > left ? left : w;
        if (p < 1024) need[p] = w;
        sum_need += w;
    }
    const double pool = (double)G->pool_tiles * kTile;
    const double scale = sum_need > pool ? pool / sum_need : 1.0;
    unsigned long long bm = 0, active = 0;
    for (int p = 0; p < n_points; ++p) {
        SweepState &S = sw[p];
        DevPoint &P = pts[p];
        P.bm_off = bm;
        if (S.done) {
            P.n = 0;
            P.n_tiles = 0;
            P.static_tiles = 0;
            continue;
        }
        P.i0 += P.n;
        const unsigned long long left = S.i_end - P.i0;
        unsigned long long w = S.window;
        if (G->adaptive && p < 1024) {
            // whole blocks of 65536 proposals, at least one, within the pool share
            const double share = need[p] * scale;
            const unsigned long long seg = 65536;
            w = (unsigned long long)(share / (double)seg) * seg;
            w = w < seg ? seg : w;
        }
        P.n = left < w ? left : w;
        P.n_tiles = (P.n + kTile - 1) / kTile;
        P.target = S.target - S.accepted;
        // dealt out evenly: three quarters of what the measured acceptance asks for
        const double used = (double)(P.i0 - S.i_start);
        P.static_tiles = static_share(
            P.n_tiles,
            S.accepted > 0 ? (unsigned long long)(0.75 / kTile * (double)P.target * used / (double)S.accepted)
                           : P.n_tiles / 4,
            n_points);
        P.capacity = S.capacity > S.written ? S.capacity - S.written : 0;
        P.out_off = S.out_off + S.written;
        bm += P.n_tiles;
        ++active;
    }
    G->active = active;
}

hipError_t launch_window_advance(DevPoint *pts, const DevCounters *cnt, const PointResult *res, SweepState *sw,
                                 int n_points, SweepGlobal *G, const unsigned long long *defer_count, hipStream_t st)
{
    hipLaunchKernelGGL(k_window_advance, dim3(1), dim3(1024), 0, st, pts, cnt, res, sw, n_points, G, defer_count);
    return hipGetLastError();
}

__global__ void k_fill_u32(uint32_t *p, unsigned long long n, uint32_t v)
{
    for (unsigned long long i = (unsigned long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (unsigned long long)gridDim.x * blockDim.x)
        p[i] = v;
}

__global__ void k_bits_to_bytes(const uint32_t *bitmap, unsigned long long n, uint8_t *out)
{
    for (unsigned long long i = (unsigned long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (unsigned long long)gridDim.x * blockDim.x)
        out[i] = (uint8_t)((bitmap[i / 32] >> (i % 32)) & 1u);
}

// ---------------------------------------------------------------------------
// Host-side launchers
// ---------------------------------------------------------------------------
template <int K, int PREC, int PROP, int B = decide_block(K), int G = 1>
static hipError_t launch_decide_t(const KernelArgs &a, const int *plist, int n_plist, int n_cu,
                                  unsigned long long total_tiles, hipStream_t st, int *grid_out)
{
    constexpr int lds = decide_lds_bytes<K, PREC>() + (B / kWave) * PairCarry<3>::BYTES;
    auto kern = k_decide<K, PREC, PROP, B, G>;
    hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    int per_cu = 0;
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, B, lds);
    if (e != hipSuccess) return e;
    if (a.blocks_per_cu > 0 && a.blocks_per_cu < per_cu) per_cu = a.blocks_per_cu;
    if (per_cu < 1) per_cu = 1;
    // at least two tiles per wave (the shortest claim)
    unsigned long long want = (total_tiles + 2ull * (B / kWave) - 1) / (2ull * (B / kWave));
    unsigned long long grid = (unsigned long long)per_cu * n_cu;
    if (a.dealt) grid *= dealt_rounds(total_tiles, grid * (B / kWave));
    if (want < grid) grid = want;
    if (grid < 1) grid = 1;
    if (grid_out) *grid_out = (int)grid;
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(B), lds, st, a, plist, n_plist);
    return hipGetLastError();
}

template <int K>
static hipError_t launch_decide_k(int prec, int prop, const KernelArgs &a, const int *plist, int n_plist,
                                  int n_cu, unsigned long long tiles, hipStream_t st, int *g)
{
#define TKDV_DISPATCH_P(PR, PP) \
    if (prec == PR && prop == PP) return launch_decide_t<K, PR, PP>(a, plist, n_plist, n_cu, tiles, st, g);
    TKDV_DISPATCH_P(PREC_FP32, PROP_UNIFORM)
    TKDV_DISPATCH_P(PREC_FP32, PROP_SIGMA)
    TKDV_DISPATCH_P(PREC_BF16X3, PROP_UNIFORM)
    TKDV_DISPATCH_P(PREC_BF16X3, PROP_SIGMA)
#undef TKDV_DISPATCH_P
    return hipErrorInvalidValue;
}

template <int K, int PREC, int PROP, int B = decide_block(K), int G = 1>
static int decide_blocks_per_cu_t()
{
    constexpr int lds = decide_lds_bytes<K, PREC>() + (B / kWave) * PairCarry<3>::BYTES;
    auto kern = k_decide<K, PREC, PROP, B, G>;
    if (hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds) != hipSuccess)
        return 1;
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, B, lds) != hipSuccess) return 1;
    return per_cu < 1 ? 1 : per_cu;
}

// Tile variants of the paper's-proposal decision kernel (BF16x3 products; the
// sweep's autotuner times them).  Variant 0 is the default configuration;
// variants 1..3 at K = 16, 32, 64 (workgroup threads, tile pairs per group):
//   K = 16: (512, 1), (1024, 1), (768, 1)
//   K = 32: (512, 1), (1024, 1), (256, 2)
//   K = 64: variant 0 is the quarter-period kernel (16 proposals per wave,
//           tkdv_quarter.hip, its own tables); 1..3 the half-period k_decide
//           in (512, 1), (1024, 1), (768, 1)
//   K = 128: the quarter-period kernel in workgroups of 512, 768, 1024
// K = 8, and FP32 products, have variant 0 only.
template <int K>
struct DecideVariant;
template <>
struct DecideVariant<16> {
    static constexpr int B[4] = {decide_block(16), 512, 1024, 768}, G[4] = {1, 1, 1, 1};
};
template <>
struct DecideVariant<32> {
    static constexpr int B[4] = {decide_block(32), 512, 1024, 256}, G[4] = {1, 1, 1, 2};
};
template <>
struct DecideVariant<64> {  // B[0]: the quarter-period kernel's workgroup
    static constexpr int B[4] = {decide_block(64), 512, 1024, kHalfPeriod64Block}, G[4] = {1, 1, 1, 1};
};

template <int K, int V>
static hipError_t launch_variant_t(const KernelArgs &a, const int *plist, int n_plist, int n_cu,
                                   unsigned long long tiles, hipStream_t st, int *g)
{
    return launch_decide_t<K, PREC_BF16X3, PROP_SIGMA, DecideVariant<K>::B[V], DecideVariant<K>::G[V]>(
        a, plist, n_plist, n_cu, tiles, st, g);
}
template <int K, int V>
static int variant_blocks_per_cu_t()
{
    return decide_blocks_per_cu_t<K, PREC_BF16X3, PROP_SIGMA, DecideVariant<K>::B[V], DecideVariant<K>::G[V]>();
}

static bool has_variants(int K, int prec, int prop)
{
    return (K == 16 || K == 32 || K == 64) && prec == PREC_BF16X3 && prop == PROP_SIGMA;
}

int decide_n_variants(int K, int prec)
{
    if (prec != PREC_BF16X3) return 1;
    if (K == 128) return decide128_n_variants();
    return has_variants(K, prec, PROP_SIGMA) ? TKDV_DECIDE_VARIANTS : 1;
}

int decide_variant_block(int K, int variant)
{
    if (variant <= 0 || variant >= TKDV_DECIDE_VARIANTS) return decide_block(K);
    switch (K) {
    case 128: return decide128_variant_block(variant);
    case 16: return DecideVariant<16>::B[variant];
    case 32: return DecideVariant<32>::B[variant];
    case 64: return DecideVariant<64>::B[variant];
    default: return decide_block(K);
    }
}

hipError_t launch_decide_variant(int K, int prec, int prop, int variant, const KernelArgs &a, const int *plist,
                                 int n_plist, int n_cu, unsigned long long tiles, hipStream_t st, int *grid_out)
{
    if (K == 128 && prec == PREC_BF16X3 && prop == PROP_SIGMA && variant > 0 && variant < decide128_n_variants())
        return launch_decide128_variant(variant, a, plist, n_plist, n_cu, tiles, st, grid_out);
    if (variant <= 0 || variant >= TKDV_DECIDE_VARIANTS || !has_variants(K, prec, prop))
        return launch_decide(K, prec, prop, a, plist, n_plist, n_cu, tiles, st, grid_out);
#define TKDV_DISPATCH_V(KK)                                                                          \
    if (K == KK) {                                                                                  \
        if (variant == 1) return launch_variant_t<KK, 1>(a, plist, n_plist, n_cu, tiles, st, grid_out); \
        if (variant == 2) return launch_variant_t<KK, 2>(a, plist, n_plist, n_cu, tiles, st, grid_out); \
        return launch_variant_t<KK, 3>(a, plist, n_plist, n_cu, tiles, st, grid_out);               \
    }
    TKDV_DISPATCH_V(16) TKDV_DISPATCH_V(32) TKDV_DISPATCH_V(64)
#undef TKDV_DISPATCH_V
    return hipErrorInvalidValue;
}

int decide_variant_max_blocks_per_cu(int K, int prec, int variant)
{
    if (K == 128 && prec == PREC_BF16X3 && variant > 0 && variant < decide128_n_variants())
        return decide128_variant_max_blocks_per_cu(variant);
    if (variant <= 0 || variant >= TKDV_DECIDE_VARIANTS || !has_variants(K, prec, PROP_SIGMA))
        return decide_max_blocks_per_cu(K, prec);
#define TKDV_DISPATCH_W(KK)                                             \
    if (K == KK) {                                                     \
        if (variant == 1) return variant_blocks_per_cu_t<KK, 1>();      \
        if (variant == 2) return variant_blocks_per_cu_t<KK, 2>();      \
        return variant_blocks_per_cu_t<KK, 3>();                        \
    }
    TKDV_DISPATCH_W(16) TKDV_DISPATCH_W(32) TKDV_DISPATCH_W(64)
#undef TKDV_DISPATCH_W
    return 1;
}

int decide_max_blocks_per_cu(int K, int prec)
{
#define TKDV_DISPATCH_O(KK, PR) \
    if (K == KK && prec == PR) return decide_blocks_per_cu_t<KK, PR, PROP_SIGMA>();
    TKDV_DISPATCH_O(8, PREC_FP32) TKDV_DISPATCH_O(8, PREC_BF16X3)
    TKDV_DISPATCH_O(16, PREC_FP32) TKDV_DISPATCH_O(16, PREC_BF16X3)
    TKDV_DISPATCH_O(32, PREC_FP32) TKDV_DISPATCH_O(32, PREC_BF16X3)
#undef TKDV_DISPATCH_O
    if (K == 64) return decide_quarter64_max_blocks_per_cu(prec);
    if (K == 128) return decide128_max_blocks_per_cu(prec);
    return 1;
}

hipError_t launch_decide(int K, int prec, int prop, const KernelArgs &a, const int *plist, int n_plist,
                         int n_cu, unsigned long long tiles, hipStream_t st, int *grid_out)
{
    switch (K) {
    case 8: return launch_decide_k<8>(prec, prop, a, plist, n_plist, n_cu, tiles, st, grid_out);
    case 16: return launch_decide_k<16>(prec, prop, a, plist, n_plist, n_cu, tiles, st, grid_out);
    case 32: return launch_decide_k<32>(prec, prop, a, plist, n_plist, n_cu, tiles, st, grid_out);
    case 64: return launch_decide_quarter64(prec, prop, a, plist, n_plist, n_cu, tiles, st, grid_out);
    case 128: return launch_decide128(prec, prop, a, plist, n_plist, n_cu, tiles, st, grid_out);
    default: return hipErrorInvalidValue;
    }
}

template <int K, int PREC>
static hipError_t launch_decide_mix_t(const KernelArgs &a, const int *plist, int n_plist, int n_cu,
                                      unsigned long long total_tiles, hipStream_t st, int *grid_out)
{
    constexpr int lds = decide_mix_lds_bytes<K, PREC>() + (kMixBlock / kWave) * PairCarry<6>::BYTES;
    auto kern = k_decide_mix<K, PREC>;
    hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    int per_cu = 0;
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, kMixBlock, lds);
    if (e != hipSuccess) return e;
    if (a.blocks_per_cu > 0 && a.blocks_per_cu < per_cu) per_cu = a.blocks_per_cu;
    if (per_cu < 1) per_cu = 1;
    unsigned long long want = (total_tiles + 2ull * (kMixBlock / kWave) - 1) / (2ull * (kMixBlock / kWave));
    unsigned long long grid = (unsigned long long)per_cu * n_cu;
    if (want < grid) grid = want;
    if (grid < 1) grid = 1;
    if (grid_out) *grid_out = (int)grid;
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(kMixBlock), lds, st, a, plist, n_plist);
    return hipGetLastError();
}

hipError_t launch_decide_mix(int K, int prec, const KernelArgs &a, const int *plist, int n_plist, int n_cu,
                             unsigned long long tiles, hipStream_t st, int *grid_out)
{
#define TKDV_DISPATCH_X(KK, PR) \
    if (K == KK && prec == PR) return launch_decide_mix_t<KK, PR>(a, plist, n_plist, n_cu, tiles, st, grid_out);
    TKDV_DISPATCH_X(8, PREC_FP32) TKDV_DISPATCH_X(8, PREC_BF16X3)
    TKDV_DISPATCH_X(16, PREC_FP32) TKDV_DISPATCH_X(16, PREC_BF16X3)
    TKDV_DISPATCH_X(32, PREC_FP32) TKDV_DISPATCH_X(32, PREC_BF16X3)
#undef TKDV_DISPATCH_X
    return hipErrorInvalidValue;
}

hipError_t launch_fixup_mix(int K, const KernelArgs &a, bool plan, int n_cu, hipStream_t st)
{
    const dim3 g(8 * n_cu), b(kBlock);
    switch (K) {
    case 8: hipLaunchKernelGGL(k_fixup_mix<8>, g, b, 0, st, a, plan ? 1 : 0); break;
    case 16: hipLaunchKernelGGL(k_fixup_mix<16>, g, b, 0, st, a, plan ? 1 : 0); break;
    case 32: hipLaunchKernelGGL(k_fixup_mix<32>, g, b, 0, st, a, plan ? 1 : 0); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_fixup(int K, const KernelArgs &a, bool plan, int n_cu, hipStream_t st)
{
    const dim3 g(4 * n_cu), b(kBlock);
    switch (K) {
    case 8: hipLaunchKernelGGL(k_fixup<8>, g, b, 0, st, a, plan ? 1 : 0); break;
    case 16: hipLaunchKernelGGL(k_fixup<16>, g, b, 0, st, a, plan ? 1 : 0); break;
    case 32: hipLaunchKernelGGL(k_fixup<32>, g, b, 0, st, a, plan ? 1 : 0); break;
    case 64: hipLaunchKernelGGL(k_fixup<64>, g, b, 0, st, a, plan ? 1 : 0); break;
    case 128: hipLaunchKernelGGL(k_fixup<128>, g, b, 0, st, a, plan ? 1 : 0); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_segments(const KernelArgs &a, unsigned long long n_segs_max, int n_cu, hipStream_t st)
{
    unsigned long long g = (n_segs_max + kBlock / kWave - 1) / (kBlock / kWave);
    if (g > 8ull * n_cu) g = 8ull * n_cu;
    hipLaunchKernelGGL(k_seg_count, dim3((unsigned)g), dim3(kBlock), 0, st, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_seg_scan, dim3(1), dim3(1024), 0, st, a);
    return hipGetLastError();
}

template <int K, int PROP>
static hipError_t launch_materialize_t(const KernelArgs &a, unsigned long long n_runs_max, float *out_xhat,
                                       unsigned long long *out_index, int n_cu, hipStream_t st)
{
    constexpr int lds = materialize_lds_bytes<K>();
    auto kern = k_materialize<K, PROP>;
    hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    unsigned long long g = (n_runs_max + kBlock / kWave - 1) / (kBlock / kWave);
    if (g > 8ull * n_cu) g = 8ull * n_cu;
    if (g < 1) g = 1;
    hipLaunchKernelGGL(kern, dim3((unsigned)g), dim3(kBlock), lds, st, a, out_xhat, out_index);
    return hipGetLastError();
}

hipError_t launch_materialize(int K, int prop, const KernelArgs &a, unsigned long long n_runs_max, float *out_xhat,
                              unsigned long long *out_index, int n_cu, hipStream_t st)
{
    if (K == 64 || K == 128) return launch_materialize_quarter(K, prop, a, n_runs_max, out_xhat, out_index, n_cu, st);
#define TKDV_DISPATCH_M(KK, PP) \
    if (K == KK && prop == PP) return launch_materialize_t<KK, PP>(a, n_runs_max, out_xhat, out_index, n_cu, st);
    TKDV_DISPATCH_M(8, PROP_UNIFORM)
    TKDV_DISPATCH_M(8, PROP_SIGMA)
    TKDV_DISPATCH_M(16, PROP_UNIFORM)
    TKDV_DISPATCH_M(16, PROP_SIGMA)
    TKDV_DISPATCH_M(32, PROP_UNIFORM)
    TKDV_DISPATCH_M(32, PROP_SIGMA)
    TKDV_DISPATCH_M(8, PROP_MIXTURE)
    TKDV_DISPATCH_M(16, PROP_MIXTURE)
    TKDV_DISPATCH_M(32, PROP_MIXTURE)
#undef TKDV_DISPATCH_M
    return hipErrorInvalidValue;
}

hipError_t launch_finalize(const KernelArgs &a, hipStream_t st)
{
    hipLaunchKernelGGL(k_finalize, dim3(a.n_points), dim3(kFinBlock), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_fill_u32(void *p, unsigned long long n_words, uint32_t v, hipStream_t st)
{
    if (n_words == 0) return hipSuccess;
    unsigned long long g = (n_words + kBlock - 1) / kBlock;
    if (g > 4096) g = 4096;
    hipLaunchKernelGGL(k_fill_u32, dim3((unsigned)g), dim3(kBlock), 0, st, (uint32_t *)p, n_words, v);
    return hipGetLastError();
}

hipError_t launch_bits_to_bytes(const uint32_t *bitmap, unsigned long long n, uint8_t *out, hipStream_t st)
{
    if (n == 0) return hipSuccess;
    unsigned long long g = (n + kBlock - 1) / kBlock;
    if (g > 4096) g = 4096;
    hipLaunchKernelGGL(k_bits_to_bytes, dim3((unsigned)g), dim3(kBlock), 0, st, bitmap, n, out);
    return hipGetLastError();
}

}  // namespace tkdv
