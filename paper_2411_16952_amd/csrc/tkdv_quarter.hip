// Quarter-period kernels of the TKdV rejection sampler at K = 64 and 128
// (N = 256, 512): the decision kernel, the ordered output with the
// statistics, and the standalone synthesis at K = 128.  The layout and the quarter-period synthesis are described
// in tkdv_quarter.h.
#include <hip/hip_runtime.h>

#include "tkdv_device.h"
#include "tkdv_kernels.h"
#include "tkdv_quarter.h"

namespace tkdv {

namespace {

// Bytes of LDS a wave of k_decide128 carries from tile to tile: three values of 64 proposals.
constexpr int kCarry128 = 3 * kWave * 4;

// ---------------------------------------------------------------------------
// k_decide128: per wave, up to 64 accept words at a time (2048 proposals, 128 tiles
// of 16), dealt out or claimed from per-point queues as in the other decision kernels.
// ---------------------------------------------------------------------------
// DBG: the verification entry's instantiation (per-proposal outputs written,
// workgroups of Quarter<K>::BLOCK); the sampling calls run the one without,
// which needs fewer registers.  BL: workgroup threads (decide_block(K), or a
// tile variant's).  |X| and t are finished before the synthesis: left for
// after it, the compiler keeps the sin block's 32 coordinates (K = 128) live
// through the products to sum their squares there, which leaves room for 2
// waves per SIMD instead of 3.
template <int K, int PREC, int PROP, bool DBG, int BL = decide_block(K)>
__global__ void __launch_bounds__(BL) k_decide128(KernelArgs a, const int *plist, int n_plist)
{
    if (a.d_active && *a.d_active == 0ull) return;  // a sweep window without unfinished points
    extern __shared__ __attribute__((aligned(16))) char lds[];
    __shared__ DeferList deferred;
    deferred.begin();
    constexpr int B = BL, CPL = K / 4;
    {
        const uint4 *s0 = reinterpret_cast<const uint4 *>(a.phi_hi);
        const uint4 *s1 = reinterpret_cast<const uint4 *>(a.phi_lo);
        uint4 *d = reinterpret_cast<uint4 *>(lds);
        constexpr int one = (PREC == PREC_FP32 ? Quarter<K>::F32_BYTES : Quarter<K>::BF16_BYTES) / 16;
        for (int v = threadIdx.x; v < one; v += B) d[v] = s0[v];
        if constexpr (PREC == PREC_BF16X3)
            for (int v = threadIdx.x; v < one; v += B) d[one + v] = s1[v];
    }
    __syncthreads();
    const char *lds_hi = lds;
    const char *lds_lo = lds + (PREC == PREC_FP32 ? 0 : Quarter<K>::BF16_BYTES);
    const int lane = threadIdx.x & 63, g = lane >> 4, pl = lane & 15;
    const unsigned gwave = __builtin_amdgcn_readfirstlane(blockIdx.x * (B / kWave) + (threadIdx.x >> 6));
    const unsigned W = gridDim.x * (B / kWave);
    const float share = (float)n_plist / (2.0f * (float)W);
    PointTally tally;
    float *carry = reinterpret_cast<float *>(lds + Quarter<K>::lds(PREC)) + (threadIdx.x >> 6) * (kCarry128 / 4);
    WaveWork<K> work(gwave, n_plist);
    unsigned long long base;
    int len;
    while (work.next(a, plist, n_plist, gwave, W, share, lane, tally, base, len)) {
        const int p = __builtin_amdgcn_readfirstlane(work.p);
        const DevPoint &P = a.pts[p];
        DevCounters *C = a.cnt + p;
        // accept bits and FP64 bits of word `lane` of this claim
        uint32_t my_word = 0u, my_def = 0u;
        const int tiles = (2 * len + 3) & ~3;  // groups of four tiles: two accept words
        const unsigned long long stop = claim_stop(P, base, len);
#pragma unroll 1
        for (int c2 = 0; c2 < tiles; ++c2) {
            asm volatile("" ::: "memory");  // as in k_decide: no hoisting of the constants
            const unsigned long long first = (base + (c2 >> 1)) * kTile + (c2 & 1) * kTile16;  // the tile's first proposal
            const uint64_t i = P.i0 + first + pl;
            if (DBG && a.dbg_xhat) {  // verification: the projected point, generated once more
                float c[CPL], s[CPL], tt;
                gen_x128<K, PROP, true, true>(P, i, g, c, s, tt);  // the decision's draw
                if (first + pl < stop) {
                    float *row = a.dbg_xhat + (first + pl) * (2 * K);
#pragma unroll
                    for (int j = 0; j < CPL; ++j) {
                        row[CPL * g + j] = c[j];
                        row[K + CPL * g + j] = s[j];
                    }
                }
            }
            const uint32_t c0 = (uint32_t)i, c1 = (uint32_t)(i >> 32);
            float r2 = 0.0f, a1 = 0.0f, a2 = 0.0f, s3l;
            float *mine = carry + (c2 & 3) * kTile16 + pl;  // this tile's |X|^2, sum k^2 X_k^2 and S3
            auto norms = [&]() {
                const float tk = weighted_part128<K>(g, r2, a1, a2);
                const float r2s = sum4(r2), tks = sum4(tk);
                if (g == 0) {
                    mine[0] = r2s;
                    mine[kWave] = tks;
                }
                __builtin_amdgcn_sched_barrier(0);
            };
            if constexpr (PREC == PREC_FP32) {
                float c[CPL], s[CPL];
                gen_block128<K, PROP>(P, c0, c1, g, 0, c, r2, a1, a2);
                gen_block128<K, PROP>(P, c0, c1, g, 1, s, r2, a1, a2);
                norms();
                s3l = cube_sum_q128_f32<K>(c, s, lds_hi, lane);
            } else {
                // one block at a time: its coordinates die once split into operands
                constexpr int R = Quarter<K>::STEPS;
                bf16x8 bh[4][R], bl[4][R];
#pragma unroll
                for (int blk = 0; blk < 2; ++blk) {
                    float v[CPL];
                    gen_block128<K, PROP>(P, c0, c1, g, blk, v, r2, a1, a2);
#pragma unroll
                    for (int odd = 0; odd < 2; ++odd)
#pragma unroll
                        for (int r = 0; r < R; ++r)
                            quarter_operand<CPL, PREC == PREC_BF16X3>(v, odd, r, bh[2 * blk + odd][r],
                                                                      bl[2 * blk + odd][r]);
                    // keep the next block's generation after this split (register pressure)
                    __builtin_amdgcn_sched_barrier(0);
                }
                norms();
                s3l = cube_sum_q128_bf16<K, PREC, K == 128 ? 2 : 1>(bh, bl, lds_hi, lds_lo, lane);
            }
            s3l = sum4(s3l);
            if (g == 0) mine[2 * kWave] = s3l;
            if ((c2 & 3) != 3) continue;
            // settle four tiles at once, a proposal per lane: lane l takes proposal
            // 16 (c2 - 3) + l of the claim (one acceptance word, log a and verdict for
            // each proposal instead of four).  Four points of 6e7 at K = 64 and 128: 42.4 -> 41.4 ms
            wave_lds_sync();
            const float inv = __builtin_amdgcn_rsqf(carry[lane]);
            const float t = carry[kWave + lane] * (inv * inv);
            const float s3 = carry[2 * kWave + lane] * (inv * inv * inv);
            wave_lds_sync();
            const unsigned long long local = first - 3 * kTile16 + lane;
            const bool valid = local < stop;
            const uint32_t w_acc = acceptance_word<K>(P, P.i0 + local);
            const float la = log_a_f32<PROP>(P, t, s3);
            bool accept, defer;
            verdict(P, la, w_acc, valid, accept, defer);
            const unsigned long long bacc = __ballot(accept);
            const unsigned long long bdef = __ballot(defer);
            const bool word = (lane & ~1) == ((c2 >> 1) & ~1);  // lanes of the group's two accept words
            if (word) my_word = (uint32_t)((lane & 1) ? bacc >> 32 : bacc);
            if (bdef) {
                if (word) my_def = (uint32_t)((lane & 1) ? bdef >> 32 : bdef);
            }
            if (valid) {
                tally.n_viol += (la > 0.0f && !defer) ? 1u : 0u;  // window proposals: k_fixup
                tally.max_la = fmaxf(tally.max_la, la);
                if (DBG && a.dbg_t) {
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
    deferred.flush(a);
}

// ---------------------------------------------------------------------------
// k_materialize_q: the ordered output and the statistics at K = 64 and 128.
// A wave takes one run of ranks at a time (RankReader), its accepted proposals
// in chunks of 16 (the decision kernel's layout), regenerated with the decision
// kernel's arithmetic and written at their rank.  The grid values come from the
// quarter-period form on the statistics grid xi_j = -pi + 2 pi j/N itself:
// representatives xi_rho = 2 pi rho/N, rho < K (FP32 16x16x4 products, table
// in LDS, entries unscaled), each giving u at xi, -xi, pi - xi and xi - pi
// from Ce, Co, Se, So; rho = 0 has only the two points 0 and pi, and the
// points +-pi/2 (rho = K) come from direct sums: cos(k pi/2) and sin(k pi/2)
// are 0 or +-1.  Full chunks only are regenerated (but for a run's last): at an
// acceptance of 1e-3 a group of 32 accept words holds one accepted proposal.
// Bound by the draw (VALU) and the FP32 products (matrix cores), which waves of
// a SIMD overlap: four points of 6e7 proposals at K = 64 and 128, 6.5e7
// accepted, 31.6 ms with ten FP64 operations and two counters a grid value,
// three waves per SIMD at K = 64 and long segments of accept words; now 24.0.
// ---------------------------------------------------------------------------
template <int K>
struct MatQ {
    static constexpr int W = 8;                      // waves per workgroup
    static constexpr int GROUP = 32;                 // words per group (lanes 0..31)
    using Ranks = RankReader<GROUP, kTile16>;
    static constexpr int LIST_BYTES = W * Ranks::N * 2;
    static constexpr int LDS = Quarter<K>::F32_BYTES + LIST_BYTES;
};

template <int K, int PROP>
__global__ void __launch_bounds__(MatQ<K>::W * kWave) k_materialize_q(KernelArgs a, float *out_xhat,
                                                                      unsigned long long *out_index)
{
    constexpr int W = MatQ<K>::W, B = W * kWave, CPL = K / 4, QG = Quarter<K>::QG;
    extern __shared__ __attribute__((aligned(16))) char lds[];
    __shared__ unsigned int wave_hist[W][kNBins];
    const unsigned long long total = cut_first(a.runs, a.n_points);
    if ((unsigned long long)blockIdx.x * W >= total) return;
    {
        const uint4 *s0 = reinterpret_cast<const uint4 *>(a.phi_hi);
        uint4 *d = reinterpret_cast<uint4 *>(lds);
        for (int v = threadIdx.x; v < Quarter<K>::F32_BYTES / 16; v += B) d[v] = s0[v];
    }
    const float4 *tab = reinterpret_cast<const float4 *>(lds);
    const int lane = threadIdx.x & 63, g = lane >> 4, pl = lane & 15;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint16_t *mylist = reinterpret_cast<uint16_t *>(lds + Quarter<K>::F32_BYTES) + wv * MatQ<K>::Ranks::N;
    WaveHist hist;
    hist.bins = wave_hist[wv];
    __syncthreads();
    const unsigned long long waves = (unsigned long long)gridDim.x * W;
    for (unsigned long long run = (unsigned long long)blockIdx.x * W + wv; run < total; run += waves) {
        const int p = __builtin_amdgcn_readfirstlane(point_of_cut(a.runs, a.n_points, run, lane));
        const DevPoint &P = a.pts[p];
        if (P.K != K || P.proposal != PROP) continue;
        hist.enter(a, p, lane);
        const PointRanks &R = a.ranks[p];
        const int sh = cut_shift(a.runs, p);
        const unsigned long long first = (run - cut_first(a.runs, p)) << sh, n = R.samples;
        typename MatQ<K>::Ranks ranks(a, R, P.bm_off, mylist, first, n - first < (1ull << sh) ? n : first + (1ull << sh),
                                      lane);
        GridSums sums;
        unsigned int n_max4 = 0;
        unsigned long long peak_idx = ~0ull;
        unsigned int peak_key = 0u;
        while (const int upto = ranks.next(lane)) {
            for (int c0 = 0; c0 < upto; c0 += kTile16) {
                const bool valid = c0 + pl < upto;
                const uint64_t i = P.i0 + (valid ? ranks.local(c0 + pl) : 0ull);
                const unsigned long long r = ranks.rank + c0 + pl;
                float c[CPL], s[CPL], t;
                gen_x128<K, PROP, true>(P, i, g, c, s, t);
                if (valid && r < P.capacity) {
                    if (out_xhat) {
                        float *row = out_xhat + (P.out_off + r) * P.row_stride;
#pragma unroll
                        for (int j = 0; j < CPL; ++j) {
                            row[CPL * g + j] = c[j];
                            row[K + CPL * g + j] = s[j];
                        }
                    }
                    if (out_index && g == 0) out_index[P.out_off + r] = i;
                }
                if (valid && g == 0 && r + 1 == P.target) a.cnt[p].last_index = i;
                if (__any(!valid)) {  // no sample, no contribution: u~ = 0
#pragma unroll
                    for (int j = 0; j < CPL; ++j) {
                        c[j] = valid ? c[j] : 0.0f;
                        s[j] = valid ? s[j] : 0.0f;
                    }
                }
                sums.umax = -INFINITY;
#pragma unroll 1
                for (int tau = 0; tau < Quarter<K>::TILES; ++tau) {
                    f32x4 acc[4] = {f32x4{}, f32x4{}, f32x4{}, f32x4{}};
#pragma unroll
                    for (int q4 = 0; q4 < QG; ++q4)
#pragma unroll
                        for (int o = 0; o < 4; ++o) {
                            // out o: 0 Ce, 1 Co, 2 Se, 3 So; coordinate 2 idx + 1 (even mode) or 2 idx (odd)
                            const float4 av = tab[((tau * 4 + o) * QG + q4) * 64 + lane];
                            const float *v = (o < 2) ? c : s;
                            const int par = (o == 0 || o == 2) ? 1 : 0;
                            acc[o] = __builtin_amdgcn_mfma_f32_16x16x4f32(av.x, v[2 * (4 * q4 + 0) + par], acc[o], 0, 0, 0);
                            acc[o] = __builtin_amdgcn_mfma_f32_16x16x4f32(av.y, v[2 * (4 * q4 + 1) + par], acc[o], 0, 0, 0);
                            acc[o] = __builtin_amdgcn_mfma_f32_16x16x4f32(av.z, v[2 * (4 * q4 + 2) + par], acc[o], 0, 0, 0);
                            acc[o] = __builtin_amdgcn_mfma_f32_16x16x4f32(av.w, v[2 * (4 * q4 + 3) + par], acc[o], 0, 0, 0);
                        }
                    float u[16];
#pragma unroll
                    for (int v = 0; v < 4; ++v) {  // representative rho = 16 tau + 4 g + v
                        const float pe = acc[0][v] + acc[1][v], me = acc[0][v] - acc[1][v];
                        const float ps = acc[2][v] + acc[3][v], ms = acc[2][v] - acc[3][v];
                        u[4 * v] = pe + ps;      // xi
                        u[4 * v + 1] = me + ms;  // xi - pi
                        u[4 * v + 2] = pe - ps;  // -xi
                        u[4 * v + 3] = me - ms;  // pi - xi
                    }
                    // rho = 0: xi = 0 and pi only (u has mean 0, so its largest value is not below the 0)
                    const bool twice = tau == 0 && g == 0;
                    u[2] = twice ? 0.0f : u[2];
                    u[3] = twice ? 0.0f : u[3];
                    sums.add(u);
                }
                // xi = +-pi/2: A = sum_k a_k cos(k pi/2), B = sum_k b_k sin(k pi/2); mode
                // K g/4 + j + 1 is j + 1 modulo 4
                float Av = 0.0f, Bv = 0.0f;
#pragma unroll
                for (int j = 0; j < CPL; j += 4) {
                    Av += c[j + 3] - c[j + 1];
                    Bv += s[j] - s[j + 2];
                }
                Av = sum4(Av);
                Bv = sum4(Bv);
                {
                    const float u[2] = {g == 0 ? Av + Bv : 0.0f, g == 0 ? Av - Bv : 0.0f};
                    sums.add(u);
                }
                // the proposal's grid values are split over lanes l, l ^ 16, l ^ 32, l ^ 48
                float umax = fmaxf(sums.umax, __shfl_xor(sums.umax, 16, 64));
                umax = fmaxf(umax, __shfl_xor(umax, 32, 64));
                // u(0) = sqrt(2 E0/pi) sum_k x^_k; bin of u(0)/u_max = sum_k x^_k / sqrt(K)
                double s0 = 0.0;
#pragma unroll
                for (int j = 0; j < CPL; ++j) s0 += (double)c[j];
                s0 += __shfl_xor(s0, 16, 64);
                s0 += __shfl_xor(s0, 32, 64);
                if (valid && g == 0) {
                    n_max4 += umax > kFourSigmaT ? 1u : 0u;
                    peak_merge(peak_key, peak_idx, float_key(umax), i);
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

// ---------------------------------------------------------------------------
// k_synth_q: the standalone synthesis (rows of x^ in HBM -> S3 = sum of the
// cubes of the grid values of each row) at K = 128, in the quarter-period form
// on the grid offset by half a step, whose trapezoid sum of u~^3 equals that on
// xi_j = -pi + 2 pi j/N (both are exact for N >= 3K + 1), with the decision
// kernel's tables and arithmetic.
// ---------------------------------------------------------------------------  Sixteen
// rows per wave: lane l holds coordinates K/4 (l/16) .. K/4 (l/16) + K/4 - 1 of
// both blocks of row l % 16 (the column operand of the 16x16 products); the
// BF16 paths split each block into operands as it arrives.  Workgroups of
// Quarter<K>::BLOCK threads share the tables (128 KB for FP32 and BF16x3).
template <int K, int PREC>
__global__ void __launch_bounds__(Quarter<K>::BLOCK) k_synth_q(const float *__restrict__ xhat, unsigned long long n,
                                                               float *__restrict__ s3_out, const void *phi_hi,
                                                               const void *phi_lo)
{
    constexpr int B = Quarter<K>::BLOCK, CPL = K / 4, R = Quarter<K>::STEPS;
    constexpr int one = (PREC == PREC_FP32 ? Quarter<K>::F32_BYTES : Quarter<K>::BF16_BYTES) / 16;
    extern __shared__ __attribute__((aligned(16))) char lds[];
    {
        const uint4 *s0 = reinterpret_cast<const uint4 *>(phi_hi);
        const uint4 *s1 = reinterpret_cast<const uint4 *>(phi_lo);
        uint4 *d = reinterpret_cast<uint4 *>(lds);
        for (int v = threadIdx.x; v < one; v += B) d[v] = s0[v];
        if constexpr (PREC == PREC_BF16X3)
            for (int v = threadIdx.x; v < one; v += B) d[one + v] = s1[v];
    }
    __syncthreads();
    const char *lds_hi = lds, *lds_lo = lds + (PREC == PREC_BF16X3 ? one * 16 : 0);
    const int lane = threadIdx.x & 63, g = lane >> 4, pl = lane & 15;
    const unsigned long long n_chunks = (n + 15) / 16;
    const unsigned long long waves = (unsigned long long)gridDim.x * (B / kWave);
    for (unsigned long long ch = (unsigned long long)blockIdx.x * (B / kWave) + (threadIdx.x >> 6); ch < n_chunks;
         ch += waves) {
        const unsigned long long row = ch * 16 + pl;
        const bool valid = row < n;
        const float *src = xhat + (valid ? row : 0ull) * (2 * K) + CPL * g;
        auto load = [&](int blk, float (&v)[CPL]) {
            const float4 *p = reinterpret_cast<const float4 *>(src + blk * K);
#pragma unroll
            for (int q = 0; q < CPL / 4; ++q) {
                const float4 w = p[q];
                v[4 * q + 0] = w.x;
                v[4 * q + 1] = w.y;
                v[4 * q + 2] = w.z;
                v[4 * q + 3] = w.w;
            }
        };
        float s3l;
        if constexpr (PREC == PREC_FP32) {
            float c[CPL], s[CPL];
            load(0, c);
            load(1, s);
            s3l = cube_sum_q128_f32<K>(c, s, lds_hi, lane);
        } else {
            bf16x8 bh[4][R], bl[4][R];
#pragma unroll
            for (int blk = 0; blk < 2; ++blk) {
                float v[CPL];
                load(blk, v);
#pragma unroll
                for (int odd = 0; odd < 2; ++odd)
#pragma unroll
                    for (int r = 0; r < R; ++r)
                        quarter_operand<CPL, PREC == PREC_BF16X3>(v, odd, r, bh[2 * blk + odd][r], bl[2 * blk + odd][r]);
            }
            s3l = cube_sum_q128_bf16<K, PREC>(bh, bl, lds_hi, lds_lo, lane);
        }
        const float s3 = sum4(s3l);
        if (valid && g == 0) s3_out[row] = s3;
    }
}

template <int K, int PREC>
hipError_t launch_synth_q_t(const float *xhat, unsigned long long n, float *s3, const void *phi_hi,
                            const void *phi_lo, int n_cu, hipStream_t st, hipEvent_t ev_start, int *grid_out,
                            int *block_out)
{
    constexpr int B = Quarter<K>::BLOCK;
    constexpr int lds = PREC == PREC_FP32 ? Quarter<K>::F32_BYTES
                                          : (PREC == PREC_BF16X3 ? 2 : 1) * Quarter<K>::BF16_BYTES;
    auto kern = k_synth_q<K, PREC>;
    hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    int per_cu = 0;
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, B, lds);
    if (e != hipSuccess) return e;
    if (per_cu < 1) per_cu = 1;
    const unsigned long long chunks = (n + 15) / 16;
    unsigned long long grid = (unsigned long long)per_cu * n_cu;
    const unsigned long long want = (chunks + B / kWave - 1) / (B / kWave);
    if (want < grid) grid = want;
    if (grid < 1) grid = 1;
    if (grid_out) *grid_out = (int)grid;
    if (block_out) *block_out = B;
    if (ev_start) {
        e = hipEventRecord(ev_start, st);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(B), lds, st, xhat, n, s3, phi_hi, phi_lo);
    return hipGetLastError();
}

template <int K, int PROP>
hipError_t launch_materialize_q_t(const KernelArgs &a, unsigned long long n_runs_max, float *out_xhat,
                                  unsigned long long *out_index, int n_cu, hipStream_t st)
{
    constexpr int lds = MatQ<K>::LDS, B = MatQ<K>::W * kWave;
    auto kern = k_materialize_q<K, PROP>;
    hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    int per_cu = 0;
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, B, lds);
    if (e != hipSuccess) return e;
    if (per_cu < 1) per_cu = 1;
    // several rounds of workgroups, so that they even out among the CUs: with one
    // round a wave's parts of a dense and of a sparse point add up or not by
    // chance (26.0 ms; 25.0 in four or eight)
    unsigned long long g = 8ull * per_cu * n_cu;
    const unsigned long long want = (n_runs_max + MatQ<K>::W - 1) / MatQ<K>::W;
    if (want < g) g = want;
    if (g < 1) g = 1;
    hipLaunchKernelGGL(kern, dim3((unsigned)g), dim3(B), lds, st, a, out_xhat, out_index);
    return hipGetLastError();
}

template <int K, int PREC, int PROP, int BL = decide_block(K)>
hipError_t launch_decide128_t(const KernelArgs &a, const int *plist, int n_plist, int n_cu,
                              unsigned long long total_tiles, hipStream_t st, int *grid_out)
{
    constexpr int BD = Quarter<K>::BLOCK;
    const bool dbg = a.dbg_xhat != nullptr || a.dbg_t != nullptr;
    const int B = dbg ? BD : BL, lds = Quarter<K>::lds(PREC) + B / kWave * kCarry128;
    auto kern = dbg ? k_decide128<K, PREC, PROP, true, BD> : k_decide128<K, PREC, PROP, false, BL>;
    hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    int per_cu = 0;
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, B, lds);
    if (e != hipSuccess) return e;
    if (a.blocks_per_cu > 0 && a.blocks_per_cu < per_cu) per_cu = a.blocks_per_cu;
    if (per_cu < 1) per_cu = 1;
    const unsigned long long per_block = 2ull * (B / kWave);  // at least two accept words per wave
    unsigned long long want = (total_tiles + per_block - 1) / per_block;
    unsigned long long grid = (unsigned long long)per_cu * n_cu;
    if (a.dealt) grid *= dealt_rounds(total_tiles, grid * (B / kWave));
    if (want < grid) grid = want;
    if (grid < 1) grid = 1;
    if (grid_out) *grid_out = (int)grid;
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(B), lds, st, a, plist, n_plist);
    return hipGetLastError();
}

template <int K, int PREC, int PROP, int BL = decide_block(K)>
int blocks_per_cu128_t()
{
    constexpr int lds = Quarter<K>::lds(PREC) + BL / kWave * kCarry128;
    auto kern = k_decide128<K, PREC, PROP, false, BL>;
    if (hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds) != hipSuccess)
        return 1;
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, BL, lds) != hipSuccess) return 1;
    return per_cu < 1 ? 1 : per_cu;
}

// Tile variants at K = 128 (BF16x3, the paper's proposal): workgroups of 768
// threads (the default: 3 waves per SIMD, no register spills), 512 (2 waves
// per SIMD) and 1024 (4 waves per SIMD, some 13 registers spilled).
constexpr int kVariants128 = 3;
constexpr int kVariant128Block[kVariants128] = {decide_block(128), 512, 1024};

template <int K>
hipError_t launch_quarter_k(int prec, int prop, const KernelArgs &a, const int *plist, int n_plist, int n_cu,
                            unsigned long long total_tiles, hipStream_t st, int *grid_out)
{
    if (prec == PREC_FP32 && prop == PROP_UNIFORM)
        return launch_decide128_t<K, PREC_FP32, PROP_UNIFORM>(a, plist, n_plist, n_cu, total_tiles, st, grid_out);
    if (prec == PREC_FP32 && prop == PROP_SIGMA)
        return launch_decide128_t<K, PREC_FP32, PROP_SIGMA>(a, plist, n_plist, n_cu, total_tiles, st, grid_out);
    if (prec == PREC_BF16X3 && prop == PROP_UNIFORM)
        return launch_decide128_t<K, PREC_BF16X3, PROP_UNIFORM>(a, plist, n_plist, n_cu, total_tiles, st,
                                                                grid_out);
    if (prec == PREC_BF16X3 && prop == PROP_SIGMA)
        return launch_decide128_t<K, PREC_BF16X3, PROP_SIGMA>(a, plist, n_plist, n_cu, total_tiles, st,
                                                              grid_out);
    return hipErrorInvalidValue;
}

}  // namespace

size_t quarter_table_bytes(int K, int prec)
{
    if (K == 64) return prec == PREC_FP32 ? Quarter<64>::F32_BYTES : Quarter<64>::BF16_BYTES;
    return prec == PREC_FP32 ? Quarter<128>::F32_BYTES : Quarter<128>::BF16_BYTES;
}

hipError_t launch_decide128(int prec, int prop, const KernelArgs &a, const int *plist, int n_plist, int n_cu,
                            unsigned long long total_tiles, hipStream_t st, int *grid_out)
{
    return launch_quarter_k<128>(prec, prop, a, plist, n_plist, n_cu, total_tiles, st, grid_out);
}

hipError_t launch_decide_quarter64(int prec, int prop, const KernelArgs &a, const int *plist, int n_plist, int n_cu,
                                   unsigned long long total_tiles, hipStream_t st, int *grid_out)
{
    return launch_quarter_k<64>(prec, prop, a, plist, n_plist, n_cu, total_tiles, st, grid_out);
}

int decide128_n_variants() { return kVariants128; }
int decide128_variant_block(int variant)
{
    return variant > 0 && variant < kVariants128 ? kVariant128Block[variant] : decide_block(128);
}

hipError_t launch_decide128_variant(int variant, const KernelArgs &a, const int *plist, int n_plist, int n_cu,
                                    unsigned long long total_tiles, hipStream_t st, int *grid_out)
{
    if (variant == 1)
        return launch_decide128_t<128, PREC_BF16X3, PROP_SIGMA, kVariant128Block[1]>(a, plist, n_plist, n_cu,
                                                                                   total_tiles, st, grid_out);
    if (variant == 2)
        return launch_decide128_t<128, PREC_BF16X3, PROP_SIGMA, kVariant128Block[2]>(a, plist, n_plist, n_cu,
                                                                                   total_tiles, st, grid_out);
    return launch_decide128_t<128, PREC_BF16X3, PROP_SIGMA>(a, plist, n_plist, n_cu, total_tiles, st, grid_out);
}

int decide128_variant_max_blocks_per_cu(int variant)
{
    if (variant == 1) return blocks_per_cu128_t<128, PREC_BF16X3, PROP_SIGMA, kVariant128Block[1]>();
    if (variant == 2) return blocks_per_cu128_t<128, PREC_BF16X3, PROP_SIGMA, kVariant128Block[2]>();
    return blocks_per_cu128_t<128, PREC_BF16X3, PROP_SIGMA>();
}

int decide128_max_blocks_per_cu(int prec)
{
    return prec == PREC_FP32 ? blocks_per_cu128_t<128, PREC_FP32, PROP_SIGMA>()
                             : blocks_per_cu128_t<128, PREC_BF16X3, PROP_SIGMA>();
}

int decide_quarter64_max_blocks_per_cu(int prec)
{
    return prec == PREC_FP32 ? blocks_per_cu128_t<64, PREC_FP32, PROP_SIGMA>()
                             : blocks_per_cu128_t<64, PREC_BF16X3, PROP_SIGMA>();
}

hipError_t launch_materialize_quarter(int K, int prop, const KernelArgs &a, unsigned long long n_runs_max,
                                      float *out_xhat, unsigned long long *out_index, int n_cu, hipStream_t st)
{
#define TKDV_DISPATCH_MQ(KK, PP) \
    if (K == KK && prop == PP) return launch_materialize_q_t<KK, PP>(a, n_runs_max, out_xhat, out_index, n_cu, st);
    TKDV_DISPATCH_MQ(64, PROP_SIGMA)
    TKDV_DISPATCH_MQ(64, PROP_UNIFORM)
    TKDV_DISPATCH_MQ(128, PROP_SIGMA)
    TKDV_DISPATCH_MQ(128, PROP_UNIFORM)
#undef TKDV_DISPATCH_MQ
    return hipErrorInvalidValue;
}

hipError_t launch_synth_quarter(int K, int prec, const float *xhat, unsigned long long n, float *s3,
                                const void *phi_hi, const void *phi_lo, int n_cu, hipStream_t st,
                                hipEvent_t ev_start, int *grid_out, int *block_out)
{
    if (K != 128) return hipErrorInvalidValue;
    if (prec == PREC_FP32)
        return launch_synth_q_t<128, PREC_FP32>(xhat, n, s3, phi_hi, phi_lo, n_cu, st, ev_start, grid_out, block_out);
    if (prec == PREC_BF16)
        return launch_synth_q_t<128, PREC_BF16>(xhat, n, s3, phi_hi, phi_lo, n_cu, st, ev_start, grid_out, block_out);
    if (prec == PREC_BF16X3)
        return launch_synth_q_t<128, PREC_BF16X3>(xhat, n, s3, phi_hi, phi_lo, n_cu, st, ev_start, grid_out,
                                                  block_out);
    return hipErrorInvalidValue;
}

}  // namespace tkdv
