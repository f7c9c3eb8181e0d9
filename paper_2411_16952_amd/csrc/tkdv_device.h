// Device building blocks of the gfx950 TKdV rejection sampler.
//
// One wavefront evaluates a tile of 32 proposals; proposal p of the tile lives
// in lanes p (cos block: coordinates x^_1..x^_K) and p + 32 (sin block:
// x^_{K+1}..x^_{2K}).  This is exactly the operand layout of the 32x32 matrix
// instructions with the proposals as the B (column) operand, so the
// spectral-to-grid synthesis u~ = Phi^T x^ needs no data movement, and each
// lane ends up holding half of its proposal's grid values.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "tkdv_internal.h"

namespace tkdv {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;

enum { PREC_FP32 = 0, PREC_BF16 = 1, PREC_BF16X3 = 2 };
enum { PROP_UNIFORM = 0, PROP_SIGMA = 1, PROP_MIXTURE = 2 };

// ---------------------------------------------------------------------------
// Philox4x32-10 (Salmon et al., SC'11): per round two 32x32->64 products of
// counter words 0 and 2 with the two multipliers, high halves XORed with the
// other counter words and the key, key advanced by the Weyl constants.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint4 philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                               uint32_t k0, uint32_t k1)
{
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        // one 32x32->64 multiply instruction per product
        const uint64_t pa = (uint64_t)c0 * 0xD2511F53u;
        const uint64_t pb = (uint64_t)c2 * 0xCD9E8D57u;
        const uint32_t hi_a = (uint32_t)(pa >> 32), lo_a = (uint32_t)pa;
        const uint32_t hi_b = (uint32_t)(pb >> 32), lo_b = (uint32_t)pb;
        uint32_t n0 = __builtin_amdgcn_bitop3_b32(hi_b, c1, k0, 0x96);  // three-way xor
        uint32_t n2 = __builtin_amdgcn_bitop3_b32(hi_a, c3, k1, 0x96);
        c0 = n0; c1 = lo_b; c2 = n2; c3 = lo_a;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return make_uint4(c0, c1, c2, c3);
}

// ---------------------------------------------------------------------------
// FP32 transforms of the 32-bit words.  U = (w + 1/2) 2^-32.
// ---------------------------------------------------------------------------
__device__ __forceinline__ float log2_hw(float x) { return __builtin_amdgcn_logf(x); }

// -2 ln U of a word, U = (w + 1/2) 2^-32, with one hardware log2:
//   U < 1/2:  log2(U) (relative accuracy of the hardware log2, |ln U| > ln 2);
//   U >= 1/2: d = 1 - U is formed exactly from ~w; for d < 2^-12 the series
//             -2 ln(1 - d) = 2d + d^2 (+ 2d^3/3 + ...: truncation below d^2/3
//             <= 2^-24/3 relative), otherwise log2(1 - d) with 1 - d rounded.
//             There the absolute error of -2 ln U is ~1e-7, and with
//             r = sqrt(-2 ln U) >= 0.022 the error of r stays below 1.4e-6.
__device__ __forceinline__ float neg2_log_u_word(uint32_t w)
{
    const float two_m32 = 2.3283064365386963e-10f;
    const bool upper = (w & 0x80000000u) != 0u;
    // q = U for U < 1/2 and q = d = 1 - U for U >= 1/2 (~w = 2^32 - 1 - w), one conversion
    const uint32_t v = w ^ (uint32_t)((int32_t)w >> 31);
    const float q = __builtin_fmaf((float)v, two_m32, 0.5f * two_m32);
    const float d = q, u = q;
    const float ser = __builtin_fmaf(d, d, d + d);
    const float lg = log2_hw(upper ? 1.0f - d : u) * -1.3862943611198906f;  // -2 ln 2
    return (upper && d < 0x1p-12f) ? ser : lg;
}

// -log2 U = (-2 ln U)/(2 ln 2) of a word, five instructions fewer than
// neg2_log_u_word with its error bound (the last bits differ): the word read
// as a signed integer s (s = w - 2^32 for w >= 2^31) gives qs = (s + 1/2) 2^-32,
// which is U below 1/2 and -(1 - U) above, both exact while |s| < 2^24, so one
// conversion yields d = |qs| without the integer fold; fract(qs) is the log's
// argument (U, or 1 - d rounded) without a subtraction and a selection; and
// the factor 2 ln 2 is left out.  For words from kSeriesWord = 2^32 - 2^20 on
// (d < 2^-12) the series -log2(1 - d) = d (1 + d/2)/ln 2, truncation below d^2/3
// relative, takes the log's place (draw_fast applies it).
constexpr uint32_t kSeriesWord = 0xFFF00000u;
__device__ __forceinline__ float signed_uniform(uint32_t w)
{
    return __builtin_fmaf((float)(int32_t)w, 2.3283064365386963e-10f, 0.5f * 2.3283064365386963e-10f);
}
__device__ __forceinline__ float neg_log2_u_signed(float qs) { return -log2_hw(__builtin_amdgcn_fractf(qs)); }
__device__ __forceinline__ float neg_log2_u_series(float qs)
{
    const float d = __builtin_fabsf(qs);
    return d * __builtin_fmaf(d, 0.72134752044448170f, 1.4426950408889634f);  // 1/(2 ln 2), 1/ln 2
}

// ln U of a word (the same arithmetic, scaled by -1/2).
__device__ __forceinline__ float log_u_word(uint32_t w) { return -0.5f * neg2_log_u_word(w); }

// One Box-Muller pair: r = sqrt(-2 ln U1), (r cos 2 pi U2, r sin 2 pi U2), for
// the kernels that write rows: the folded-word form and the unit scale, so
// that the rows' bits (and what is fitted to them, such as the learned
// proposal's networks) do not move with the decision path's choices (draw_fast).
__device__ __forceinline__ void box_muller_f32(uint32_t w1, uint32_t w2, float &z0, float &z1)
{
    const float r = __builtin_amdgcn_sqrtf(neg2_log_u_word(w1));  // argument below 45
    // U2 - 1/2 = (w2 - 2^31 + 1/2) 2^-32 in revolutions, centred on zero for
    // the hardware sin/cos; the signed integer w2 - 2^31 is formed exactly.
    const float rev = __builtin_fmaf((float)(int32_t)(w2 ^ 0x80000000u), 2.3283064365386963e-10f,
                                     1.1641532182693481e-10f);
    // sin/cos(2 pi (U2 - 1/2)) = -sin/-cos(2 pi U2)
    z0 = -r * __builtin_amdgcn_cosf(rev);
    z1 = -r * __builtin_amdgcn_sinf(rev);
}

// The same draw for the decision and weight kernels, whose FP32 values only
// steer the exact FP64 decision: r from the signed-word -log2 U1, i.e. every
// coordinate scaled by 1/sqrt(2 ln 2), a common factor that the projection onto
// the sphere removes (x^, t, S3 |x|^-3 and the mixture's ratios are invariant),
// and the angle from the signed word U2 or U2 - 1 (the same angle in
// revolutions).  Pairs (w1[q], w2[q]) -> x[2q], x[2q + 1], P pairs together: the
// series near U1 = 1 takes four instructions a pair when selected each time,
// though one pair in 4096 needs it; here the wave looks once at the largest
// word and applies it only when some lane has one (one group of eight pairs in
// eight).  Every value is the one a selection per pair gives.  Decisions of 1e9
// proposals at K = 32: 48.5 -> 46.5 ms, of the mixture 74.1 -> 72.1 ms.
template <int P>
__device__ __forceinline__ void draw_fast(const uint32_t (&w1)[P], const uint32_t (&w2)[P], float *x)
{
    float l[P];
    uint32_t m = w1[0];
#pragma unroll
    for (int q = 0; q < P; ++q) {
        l[q] = neg_log2_u_signed(signed_uniform(w1[q]));
        m = w1[q] > m ? w1[q] : m;
    }
    if (__builtin_expect(__ballot(m >= kSeriesWord) != 0ull, 0)) {
#pragma unroll
        for (int q = 0; q < P; ++q) {
            const float ser = neg_log2_u_series(signed_uniform(w1[q]));
            l[q] = w1[q] >= kSeriesWord ? ser : l[q];
        }
    }
#pragma unroll
    for (int q = 0; q < P; ++q) {
        const float r = __builtin_amdgcn_sqrtf(l[q]);
        const float rev = signed_uniform(w2[q]);
        x[2 * q] = r * __builtin_amdgcn_cosf(rev);
        x[2 * q + 1] = r * __builtin_amdgcn_sinf(rev);
    }
}

// Coordinates 4 b .. 4 b + 3 from Philox block blk0 + b, b < NB (FAST: draw_fast
// in groups of kDrawBlocks blocks).
constexpr int kDrawBlocks = 4;
template <int NB, bool FAST>
__device__ __forceinline__ void draw_blocks(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t blk0, uint32_t k0,
                                            uint32_t k1, float *x)
{
    if constexpr (FAST) {
        constexpr int G = NB < kDrawBlocks ? NB : kDrawBlocks;
        static_assert(NB % G == 0, "whole groups");
#pragma unroll
        for (int g = 0; g < NB; g += G) {
            uint32_t w1[2 * G], w2[2 * G];
#pragma unroll
            for (int b = 0; b < G; ++b) {
                const uint4 w = philox4x32_10(c0, c1, c2, blk0 + (uint32_t)(g + b), k0, k1);
                w1[2 * b] = w.x;
                w2[2 * b] = w.y;
                w1[2 * b + 1] = w.z;
                w2[2 * b + 1] = w.w;
            }
            draw_fast<2 * G>(w1, w2, x + 4 * g);
        }
    } else {
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const uint4 w = philox4x32_10(c0, c1, c2, blk0 + (uint32_t)b, k0, k1);
            box_muller_f32(w.x, w.y, x[4 * b + 0], x[4 * b + 1]);
            box_muller_f32(w.z, w.w, x[4 * b + 2], x[4 * b + 3]);
        }
    }
}

// ln(1 + y) for 0 <= y: the rounding of 1 + y is corrected to first order
// with the exact difference (1 + y) - 1 (an approximate reciprocal suffices).
__device__ __forceinline__ float log1p_f32(float y)
{
    const float u = 1.0f + y;
    const float den = u - 1.0f;
    const float lg = log2_hw(u) * 0.69314718055994531f;
    return den == 0.0f ? y : lg * (y * __builtin_amdgcn_rcpf(den));
}

// Half-wave exchange: lanes 32-63 of a and lanes 0-31 of b change places.
__device__ __forceinline__ void swap32(float &a, float &b)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    a = __uint_as_float(r[0]);
    b = __uint_as_float(r[1]);
}
// The odd rows (of 16 lanes) of a and the even rows of b change places.
__device__ __forceinline__ void swap16(float &a, float &b)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    a = __uint_as_float(r[0]);
    b = __uint_as_float(r[1]);
}
// v of lane l + 32 (mod 64)
__device__ __forceinline__ float xor32(float v)
{
    float lo = v, hi = v;
    swap32(lo, hi);  // lo: lanes 0-31 twice, hi: lanes 32-63 twice
    return (threadIdx.x & 32) ? lo : hi;
}
// Lane l and l + 32 both get v(l mod 32) + v(l mod 32 + 32).
__device__ __forceinline__ float sum32(float v)
{
    float lo = v, hi = v;
    swap32(lo, hi);
    return lo + hi;
}
// One wave's LDS copies of N values of the two tiles of a pair, N x 2 x 64 floats.
// In registers they would be live through the second tile's draw and products,
// where the decision kernels have none left.
template <int N>
struct PairCarry {
    float *buf;
    __device__ __forceinline__ void put(int n, int tile, int lane, float v) const { buf[(n * 2 + tile) * 64 + lane] = v; }
    // proposal (tile, pl): the sum over its two lanes, or its first lane's value
    __device__ __forceinline__ float sum(int n, int tile, int pl) const
    {
        const float *b = buf + (n * 2 + tile) * 64 + pl;
        return b[0] + b[32];
    }
    __device__ __forceinline__ float first(int n, int tile, int pl) const { return buf[(n * 2 + tile) * 64 + pl]; }
    static constexpr int BYTES = N * 2 * 64 * 4;
};
// LDS written by a wave's lanes, read by others of the same wave.
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// ---------------------------------------------------------------------------
// Proposal generation: the K coordinates x of this lane's block (scaled by the
// proposal's standard deviations, not projected) and the lane's parts of
// |x|^2 and sum_k k^2 x_k^2; the caller sums them over the proposal's two
// lanes and scales what it derives from x by |x|^-1.  FAST selects the
// Box-Muller form: the signed-word form (draw_fast) where the draw only feeds
// a decision or a weight, the folded-word form (box_muller_f32) where rows are
// written.
// ---------------------------------------------------------------------------
// Floats that no kernel writes while it reads them, for scalar loads: as
// ordinary memory, written to by the kernel's atomics as far as the compiler
// knows, they came through vector loads into K registers a lane (1e9 proposals
// at K = 32: 45.7 -> 45.3 ms).
typedef const __attribute__((address_space(4))) float *ConstFloats;
__device__ __forceinline__ ConstFloats const_floats(const float *p) { return (ConstFloats)(uint64_t)p; }

template <int K, int PROP, bool FAST>
__device__ __forceinline__ void gen_x_part(const DevPoint &P, uint64_t i, int half, float (&x)[K], float &r2, float &tk)
{
    draw_blocks<K / 4, FAST>((uint32_t)i, (uint32_t)(i >> 32), P.point_id, (uint32_t)(half * (K / 4)), P.key0, P.key1, x);
    if (PROP == PROP_SIGMA) {
        const ConstFloats sg = const_floats(P.sig);
#pragma unroll
        for (int j = 0; j < K; ++j) x[j] *= sg[j];
    }
    r2 = 0.0f;
    tk = 0.0f;
#pragma unroll
    for (int j = 0; j < K; ++j) {
        const float sq = x[j] * x[j];
        r2 += sq;
        tk = __builtin_fmaf((float)((j + 1) * (j + 1)), sq, tk);
    }
}

// The acceptance word of proposal i (word 2K).
template <int K>
__device__ __forceinline__ uint32_t acceptance_word(const DevPoint &P, uint64_t i)
{
    return philox4x32_10((uint32_t)i, (uint32_t)(i >> 32), P.point_id, (uint32_t)(K / 2), P.key0, P.key1).x;
}

// The projected point of proposal i (rows for the caller): x^ = x |x|^-1 and t;
// the bits do not depend on the decision path's choices (box_muller_f32).
template <int K, int PROP>
__device__ __forceinline__ void gen_xhat(const DevPoint &P, uint64_t i, int half, float (&x)[K], float &t)
{
    float r2, tk;
    gen_x_part<K, PROP, false>(P, i, half, x, r2, tk);
    const float inv = __builtin_amdgcn_rsqf(sum32(r2));
    t = sum32(tk) * (inv * inv);
#pragma unroll
    for (int j = 0; j < K; ++j) x[j] *= inv;
}

// ---------------------------------------------------------------------------
// Synthesis tables in LDS.
//   BF16: [T = K/8 grid tiles][S = K/8 k-steps][64 lanes][8] bf16, hi and lo;
//         lane l, tile t, step s holds Phi(block l/32, modes 8s+1..8s+8) at
//         grid point 32t + l%32.
//   FP32: [T][Q = K/4][64][4] floats; lane l holds Phi(block l/32, modes
//         4q+1..4q+4) at grid point 32t + l%32.
// ---------------------------------------------------------------------------
template <int K>
__host__ __device__ constexpr int bf16_table_bytes() { return (K / 8) * (K / 8) * kWave * 16; }
template <int K>
__host__ __device__ constexpr int f32_table_bytes() { return (K / 8) * (K / 4) * kWave * 16; }

// BF16 operands of this lane's coordinates: hi = RNE(x), lo = RNE(x - hi).
template <int K, int PREC>
__device__ __forceinline__ void split_bf16(const float (&x)[K], bf16x8 (&bh)[K / 8], bf16x8 (&bl)[K / 8])
{
#pragma unroll
    for (int s = 0; s < K / 8; ++s) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float v = x[8 * s + e];
            const __bf16 hv = (__bf16)v;
            bh[s][e] = hv;
            if constexpr (PREC == PREC_BF16X3) bl[s][e] = (__bf16)(v - (float)hv);
        }
    }
}

// Sum over this lane's grid values of u~^3 (u~ = unscaled synthesis), with
// the products in the requested arithmetic (FP32 reads x, BF16 reads bh/bl).
// The plain (dense) form; the kernels take it at K = 8, a single grid-tile
// group, and the half-period form below for K >= 16.
template <int K, int PREC>
__device__ __forceinline__ float cube_sum_ops(const float (&x)[K], const bf16x8 (&bh)[K / 8],
                                              const bf16x8 (&bl)[K / 8], const char *lds_hi,
                                              const char *lds_lo, int lane)
{
    float s3 = 0.0f;
    if constexpr (PREC == PREC_FP32) {
        const float4 *tab = reinterpret_cast<const float4 *>(lds_hi);
#pragma unroll
        for (int t = 0; t < K / 8; ++t) {
            f32x16 acc = {};
#pragma unroll
            for (int q = 0; q < K / 4; ++q) {
                float4 a = tab[(t * (K / 4) + q) * kWave + lane];
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.x, x[4 * q + 0], acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.y, x[4 * q + 1], acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.z, x[4 * q + 2], acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.w, x[4 * q + 3], acc, 0, 0, 0);
            }
#pragma unroll
            for (int v = 0; v < 16; ++v) s3 = __builtin_fmaf(acc[v] * acc[v], acc[v], s3);
        }
    } else {
        const bf16x8 *th = reinterpret_cast<const bf16x8 *>(lds_hi);
        const bf16x8 *tl = reinterpret_cast<const bf16x8 *>(lds_lo);
#pragma unroll
        for (int t = 0; t < K / 8; ++t) {
            f32x16 acc = {};
#pragma unroll
            for (int s = 0; s < K / 8; ++s) {
                const int idx = (t * (K / 8) + s) * kWave + lane;
                const bf16x8 ah = th[idx];
                if constexpr (PREC == PREC_BF16X3) {
                    const bf16x8 al = tl[idx];
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al, bh[s], acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bl[s], acc, 0, 0, 0);
                }
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bh[s], acc, 0, 0, 0);
            }
#pragma unroll
            for (int v = 0; v < 16; ++v) s3 = __builtin_fmaf(acc[v] * acc[v], acc[v], s3);
        }
    }
    return s3;
}

template <int K, int PREC>
__device__ __forceinline__ float synth_cube_sum(const float (&x)[K], const char *lds_hi,
                                                const char *lds_lo, int lane)
{
    bf16x8 bh[K / 8], bl[K / 8];
    if constexpr (PREC != PREC_FP32) split_bf16<K, PREC>(x, bh, bl);
    return cube_sum_ops<K, PREC>(x, bh, bl, lds_hi, lds_lo, lane);
}

// ---------------------------------------------------------------------------
// Half-period form of the synthesis (K >= 16).  Shifting the grid
// xi_j = -pi + 2 pi j/N by half a period (N/2 points, T/2 of the T = N/32
// grid tiles) multiplies mode k's cos and sin rows by (-1)^k.  With E and O
// the syntheses over the even and over the odd modes on grid tile t < T/2,
// tile t holds u~ = E + O and tile t + T/2 holds u~ = E - O, so that
//     u~(t)^3 + u~(t + T/2)^3 = 2 E (E^2 + 3 O^2):
// two products over half the modes each give both tiles, half the matrix
// work of the plain product for the same sum of cubes.
//   BF16 tables (hi, lo): fragment ((t * K/16 + s) * 2 + p) * 64 + l holds for
//   lane l the 8 entries Phi(block l/32, mode 16 s + 2 e + 2 - p) at grid
//   point 32 t + l%32 (p = 0 even modes, p = 1 odd modes), t < T/2, gathered
//   from the plain tables when a workgroup stages them.
//   FP32 table: the first T/2 grid tiles of the plain table (each FP32 matrix
//   instruction takes one mode; the parity selects the accumulator).
// ---------------------------------------------------------------------------
template <int K>
__host__ __device__ constexpr int eo_steps() { return K / 16; }  // k-steps of one parity = tile pairs

// bytes of one staged table (hi or lo)
template <int K, int PREC>
__host__ __device__ constexpr int eo_table_bytes()
{
    return (PREC == PREC_FP32 ? f32_table_bytes<K>() : bf16_table_bytes<K>()) / 2;
}

// Even-mode (p = 0) or odd-mode (p = 1) fragment from two consecutive k-step
// fragments a, b of the plain BF16 table (modes 8 s + 1 .. 8 s + 16): the even
// modes are their odd entries, the high halves of the 32-bit words.
__device__ __forceinline__ uint4 gather_parity(uint4 a, uint4 b, int p)
{
    if (p == 0)
        return make_uint4((a.x >> 16) | (a.y & 0xffff0000u), (a.z >> 16) | (a.w & 0xffff0000u),
                          (b.x >> 16) | (b.y & 0xffff0000u), (b.z >> 16) | (b.w & 0xffff0000u));
    return make_uint4((a.x & 0xffffu) | (a.y << 16), (a.z & 0xffffu) | (a.w << 16), (b.x & 0xffffu) | (b.y << 16),
                      (b.z & 0xffffu) | (b.w << 16));
}

// A workgroup of BLOCK threads permutes n_tiles row tiles of plain-layout
// BF16 fragments (tile t, k-step s: modes 8 s + 1 .. 8 s + 8) into the parity
// layout: fragment ((t * K/16 + s) * 2 + p) * 64 + l.
template <int K, int BLOCK>
__device__ __forceinline__ void stage_parity_frags(uint4 *dst, const uint4 *src, int n_tiles)
{
    constexpr int S = eo_steps<K>();
    const int n = n_tiles * (K / 8) * kWave;
    for (int v = threadIdx.x; v < n; v += BLOCK) {
        const int l = v % kWave, p = (v / kWave) % 2, s = (v / (2 * kWave)) % S, t = v / (2 * kWave * S);
        const int f = (t * (K / 8) + 2 * s) * kWave + l;  // plain fragment of k-step 2s
        dst[v] = gather_parity(src[f], src[f + kWave], p);
    }
}

// A workgroup of BLOCK threads stages the half-period tables: hi at lds, lo
// (BF16x3) at lds + eo_table_bytes.  The cube sums read tables whose odd-mode
// rows carry sqrt(3) (pair_cubes); the SIR power sums read the plain ones.
template <int K, int PREC, int BLOCK>
__device__ __forceinline__ void stage_eo_tables(char *lds, const void *phi_hi, const void *phi_lo)
{
    constexpr int tab = eo_table_bytes<K, PREC>();
    uint4 *d = reinterpret_cast<uint4 *>(lds);
    if constexpr (PREC == PREC_FP32) {
        const uint4 *s0 = reinterpret_cast<const uint4 *>(phi_hi);
        for (int v = threadIdx.x; v < tab / 16; v += BLOCK) d[v] = s0[v];
    } else {
        stage_parity_frags<K, BLOCK>(d, reinterpret_cast<const uint4 *>(phi_hi), eo_steps<K>());
        if constexpr (PREC == PREC_BF16X3)
            stage_parity_frags<K, BLOCK>(d + tab / 16, reinterpret_cast<const uint4 *>(phi_lo), eo_steps<K>());
    }
}

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

// Two floats as packed BF16: hi = RNE(v), lo = RNE(v - hi) (the subtraction
// is exact: hi is v rounded to its top 16 bits).
__device__ __forceinline__ uint32_t pack_hi(float v0, float v1)
{
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2_t){v0, v1}, bf16x2_t));
}
__device__ __forceinline__ uint32_t pack_lo(float v0, float v1, uint32_t hi)
{
    const float h0 = __uint_as_float(hi << 16), h1 = __uint_as_float(hi & 0xffff0000u);
    return pack_hi(v0 - h0, v1 - h1);
}

// This lane's operands by parity (x[j] is the coordinate of mode j + 1):
// e*[s] entry e is mode 16 s + 2 e + 2, o*[s] entry e is mode 16 s + 2 e + 1.
// BF16 products fill eh and oh only.
template <int K, int PREC>
__device__ __forceinline__ void split_eo(const float (&x)[K], bf16x8 (&eh)[K / 16], bf16x8 (&el)[K / 16],
                                         bf16x8 (&oh)[K / 16], bf16x8 (&ol)[K / 16])
{
#pragma unroll
    for (int s = 0; s < K / 16; ++s) {
        u32x4_t weh, wel, woh, wol;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const int j = 16 * s + 4 * w;
            weh[w] = pack_hi(x[j + 1], x[j + 3]);
            woh[w] = pack_hi(x[j], x[j + 2]);
            if constexpr (PREC == PREC_BF16X3) {
                wel[w] = pack_lo(x[j + 1], x[j + 3], weh[w]);
                wol[w] = pack_lo(x[j], x[j + 2], woh[w]);
            }
        }
        eh[s] = __builtin_bit_cast(bf16x8, weh);
        oh[s] = __builtin_bit_cast(bf16x8, woh);
        if constexpr (PREC == PREC_BF16X3) {
            el[s] = __builtin_bit_cast(bf16x8, wel);
            ol[s] = __builtin_bit_cast(bf16x8, wol);
        }
    }
}

// hi operands only (BF16 products)
template <int K>
__device__ __forceinline__ void split_eo_hi(const float (&x)[K], bf16x8 (&eh)[K / 16], bf16x8 (&oh)[K / 16])
{
#pragma unroll
    for (int s = 0; s < K / 16; ++s) {
        u32x4_t weh, woh;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const int j = 16 * s + 4 * w;
            weh[w] = pack_hi(x[j + 1], x[j + 3]);
            woh[w] = pack_hi(x[j], x[j + 2]);
        }
        eh[s] = __builtin_bit_cast(bf16x8, weh);
        oh[s] = __builtin_bit_cast(bf16x8, woh);
    }
}

// sum over the pair's grid values of u~^3 = 2 E (E^2 + 3 O^2), elementwise,
// from co = sqrt(3) O: the odd-mode rows of the tables these sums read carry
// the factor sqrt(3), which saves a product per grid value (the factor 2 is
// applied by the caller)
__device__ __forceinline__ float pair_cubes(const f32x16 &ce, const f32x16 &co, float s)
{
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const float e = ce[v], o = co[v];
        const float q = __builtin_fmaf(o, o, e * e);
        s = __builtin_fmaf(e, q, s);
    }
    return s;
}

// S3 over this lane's grid values in the half-period form, FP32 products; G
// tile pairs per group have their accumulators live together.  The tables are
// the S3 tables: odd-mode rows scaled by sqrt(3) (pair_cubes).
template <int K, int G>
__device__ __forceinline__ float cube_sum_eo_f32(const float (&x)[K], const char *lds, int lane)
{
    constexpr int P = eo_steps<K>();
    const float4 *tab = reinterpret_cast<const float4 *>(lds);
    float s3 = 0.0f;
#pragma unroll 1
    for (int g = 0; g < P; g += G) {
        f32x16 ce[G], co[G];
#pragma unroll
        for (int u = 0; u < G; ++u) ce[u] = co[u] = f32x16{};
#pragma unroll
        for (int q = 0; q < K / 4; ++q)
#pragma unroll
            for (int u = 0; u < G; ++u) {
                // entries 0..3: modes 4q+1 (odd), 4q+2 (even), 4q+3 (odd), 4q+4 (even)
                const float4 a = tab[((g + u) * (K / 4) + q) * kWave + lane];
                co[u] = __builtin_amdgcn_mfma_f32_32x32x2f32(a.x, x[4 * q + 0], co[u], 0, 0, 0);
                ce[u] = __builtin_amdgcn_mfma_f32_32x32x2f32(a.y, x[4 * q + 1], ce[u], 0, 0, 0);
                co[u] = __builtin_amdgcn_mfma_f32_32x32x2f32(a.z, x[4 * q + 2], co[u], 0, 0, 0);
                ce[u] = __builtin_amdgcn_mfma_f32_32x32x2f32(a.w, x[4 * q + 3], ce[u], 0, 0, 0);
            }
#pragma unroll
        for (int u = 0; u < G; ++u) s3 = pair_cubes(ce[u], co[u], s3);
    }
    return 2.0f * s3;
}

// The same with BF16 (hi) or BF16x3 (hi/lo) products from the split operands;
// the lo operands el, ol are read for BF16x3 only (null for BF16).
template <int K, int PREC, int G>
__device__ __forceinline__ float cube_sum_eo_bf16(const bf16x8 (&eh)[K / 16], const bf16x8 *el,
                                                  const bf16x8 (&oh)[K / 16], const bf16x8 *ol,
                                                  const char *lds_hi, const char *lds_lo, int lane)
{
    constexpr int P = eo_steps<K>(), S = eo_steps<K>();
    const bf16x8 *th = reinterpret_cast<const bf16x8 *>(lds_hi);
    const bf16x8 *tl = reinterpret_cast<const bf16x8 *>(lds_lo);
    float s3 = 0.0f;
#pragma unroll 1
    for (int g = 0; g < P; g += G) {
        f32x16 ce[G], co[G];
#pragma unroll
        for (int u = 0; u < G; ++u) ce[u] = co[u] = f32x16{};
#pragma unroll
        for (int s = 0; s < S; ++s)
#pragma unroll
            for (int u = 0; u < G; ++u) {
                const int idx = ((g + u) * S + s) * 2 * kWave + lane;
                const bf16x8 aeh = th[idx], aoh = th[idx + kWave];
                if constexpr (PREC == PREC_BF16X3) {
                    const bf16x8 ael = tl[idx], aol = tl[idx + kWave];
                    ce[u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ael, eh[s], ce[u], 0, 0, 0);
                    co[u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(aol, oh[s], co[u], 0, 0, 0);
                    ce[u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(aeh, el[s], ce[u], 0, 0, 0);
                    co[u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(aoh, ol[s], co[u], 0, 0, 0);
                }
                ce[u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(aeh, eh[s], ce[u], 0, 0, 0);
                co[u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(aoh, oh[s], co[u], 0, 0, 0);
            }
#pragma unroll
        for (int u = 0; u < G; ++u) s3 = pair_cubes(ce[u], co[u], s3);
    }
    return 2.0f * s3;
}

// S3 of coordinates x in the half-period form with G tile pairs per group.
template <int K, int PREC, int G>
__device__ __forceinline__ float eo_cube_sum(const float (&x)[K], const char *lds_hi, const char *lds_lo, int lane)
{
    if constexpr (PREC == PREC_FP32) {
        return cube_sum_eo_f32<K, G>(x, lds_hi, lane);
    } else {
        constexpr int S = eo_steps<K>();
        bf16x8 eh[S], oh[S];
        if constexpr (PREC == PREC_BF16X3) {
            bf16x8 el[S], ol[S];
            split_eo<K, PREC>(x, eh, el, oh, ol);
            return cube_sum_eo_bf16<K, PREC, G>(eh, el, oh, ol, lds_hi, lds_lo, lane);
        } else {
            split_eo_hi<K>(x, eh, oh);
            return cube_sum_eo_bf16<K, PREC, G>(eh, nullptr, oh, nullptr, lds_hi, lds_lo, lane);
        }
    }
}

// log a = log f/(M g) in FP32 from t and S3 = sum_j u~_j^3 (both lanes identical).
template <int PROP>
__device__ __forceinline__ float log_a_f32(const DevPoint &P, float t, float s3)
{
    float lf = __builtin_fmaf(P.neg_bp_K2, t, P.c3coef * s3);
    if (PROP == PROP_SIGMA) lf = __builtin_fmaf(P.Kf, log1p_f32(P.g_coef * t), lf);
    return lf - P.log_M;
}

// The fast path's verdict on a proposal from log a and its acceptance word:
// ln U < ln a - tau <=> U < a e^-tau (accept); within the window: FP64.
// U = (w + 1/2) 2^-32; a = 2^(la log2 e) underflows to 0 only where U > a e^tau.
// Above the bound by no more than the fast path's error (0 < log a <= tau) the
// decision and the check of eq. (M_sup) are left to the FP64 pass.
__device__ __forceinline__ void verdict(const DevPoint &P, float la, uint32_t w_acc, bool valid, bool &accept, bool &defer)
{
    const float U = __builtin_fmaf((float)w_acc, 2.3283064365386963e-10f, 1.1641532182693481e-10f);
    const float alin = __builtin_amdgcn_exp2f(la * 1.4426950408889634f);
    const float lo_edge = alin * P.e_lo, hi_edge = alin * P.e_hi;
    const bool near_bound = la > 0.0f && la <= P.tau;
    defer = valid && ((U >= lo_edge && U < hi_edge) || near_bound);
    accept = valid && U < lo_edge && !near_bound;
}

// Order-preserving map float -> uint32 for atomicMax.
__device__ __forceinline__ unsigned int float_key(float f)
{
    unsigned int u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Thresholds of the statistics in units of u~ = u / sqrt(2 E0/pi): 2 sigma and
// 4 sigma, sigma = sqrt(E0/pi), are u~ = sqrt 2 and 2 sqrt 2.
constexpr float kTwoSigmaT = 1.41421356237309515f;
constexpr float kFourSigmaT = 2.82842712474619031f;

// The better of two peaks (float_key of the value, proposal index): the larger
// value, the lower index among equal values; key 0 stands for none.
__device__ __forceinline__ void peak_merge(unsigned int &key, unsigned long long &idx, unsigned int k2,
                                           unsigned long long i2)
{
    if (k2 > key || (k2 == key && k2 != 0u && i2 < idx)) {
        key = k2;
        idx = i2;
    }
}
// The peak of the wave, in every lane (the merge is a total order).
__device__ __forceinline__ void wave_peak(unsigned int &key, unsigned long long &idx)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const unsigned int k2 = __shfl_xor(key, o, 64);
        const unsigned long long i2 = __shfl_xor(idx, o, 64);
        peak_merge(key, idx, k2, i2);
    }
}

__device__ __forceinline__ unsigned long long pack_defer(int p, uint64_t i)
{
    return ((unsigned long long)p << 40) | (unsigned long long)i;
}

// ---------------------------------------------------------------------------
// Work queues of the decision kernels
// ---------------------------------------------------------------------------
__device__ __forceinline__ unsigned long long load_relaxed(const unsigned long long *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Lane 0's value, as a wave-uniform (scalar) value.  The claim loops branch
// on it: a per-lane copy would make their exits divergent for the compiler,
// which may then split a loop so that lanes wait on a lane that has left it.
__device__ __forceinline__ unsigned long long bcast_lane0(unsigned long long v)
{
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return ((unsigned long long)hi << 32) | lo;
}

// Per-wave counter update: every lane issues the atomic (lane 0 adds its
// wave-uniform value, the others 0), see claim_tiles.
__device__ __forceinline__ void add_lane0(unsigned long long *ctr, unsigned long long v, int lane)
{
    if (bcast_lane0(v) != 0ull) atomicAdd(ctr, lane == 0 ? v : 0ull);
}

// Tiles of the point's range that are decided: the static ones and the claims.
__device__ __forceinline__ unsigned long long tiles_taken(const DevPoint &P, unsigned long long next_tile)
{
    const unsigned long long t = P.static_tiles + next_tile;
    return t < P.n_tiles ? t : P.n_tiles;
}

// A wave's even share [b, e) of point P's static tiles, W waves in all, in
// pairs of tiles (which the decision kernels settle together); the remainders
// of successive points fall to different waves.
__device__ __forceinline__ void static_range(const DevPoint &P, int p, unsigned gwave, unsigned W,
                                             unsigned long long &b, unsigned long long &e)
{
    const unsigned w = (gwave + 977u * (unsigned)p) % W;
    const unsigned n = (unsigned)P.static_tiles, n2 = (n + 1) / 2;  // at most kMaxStatic
    // wave-uniform; the quotient comes from the vector unit, so say so
    const unsigned q = __builtin_amdgcn_readfirstlane(n2 / W), r = n2 - q * W;
    const unsigned b0 = 2u * (q * w + (w < r ? w : r)), e0 = b0 + 2u * (q + (w < r ? 1u : 0u));
    b = bcast_lane0((unsigned long long)(b0 < n ? b0 : n));
    e = e0 < n ? e0 : n;
}

// Claims [b, e) from the tiles after the static ones; false when none is left
// or, in accepted-count mode, the target is met by the definite accepts of
// finished work (the target-th sample is then among the tiles taken so far).
// The length is guided by what is left: share = (points)/(2 waves) of the
// point's remaining tiles, so that the last claims are short, and at least
// kMinClaim; in accepted-count mode what is left is estimated from the
// acceptance of the finished tiles, no claim is longer than that asks for, and
// once the tiles taken should do (by four standard deviations) only every
// 32nd wave, the keepers, goes on until the target is met.
// Whether they should do a wave asks of its own shard first: 4096 waves that come
// from their even shares together and read all eight wait for each other at those
// lines (K = 16, a million near-linear samples, 178 us, now 147).  (Claims of a fixed
// 64 tiles by every wave gave a near-linear point of a million samples eight
// times the proposals it needed: K = 16, 1.0 ms of decisions.)
// Every lane issues the atomic (lane 0 adds, the others add 0) and lane 0's
// old value is taken, so no lane-divergent region sits next to the loop
// back-edge (the compiler may otherwise thread lanes 1-63 past lane 0's region
// to the broadcast and split the wave).
template <int K>
__device__ __forceinline__ bool claim_tiles(const DevPoint &P, DevCounters *C, int lane, float share, bool keeper,
                                            unsigned long long &b, unsigned long long &e)
{
    // the shortest claim: a queue hands out about 5e7 claims a second
    constexpr int kMinClaim = K == 128 ? 4 : (K == 64 ? 8 : 16);
    if (P.static_tiles >= P.n_tiles) return false;
    const unsigned long long next = P.static_tiles + bcast_lane0(load_relaxed(&C->next_tile));
    if (next >= P.n_tiles) return false;
    float rem = (float)(P.n_tiles - next);
    if (P.target != ~0ull) {
        const float nx = (float)next;
        // do the tiles taken suffice, by four standard deviations, if fin tiles had ac accepts?
        auto suffice = [&](float fin, float ac) {
            return ac >= 64.0f && (float)P.target * (fin / ac) * (1.0f + 4.0f * __builtin_amdgcn_rsqf(ac)) <= nx;
        };
        if (!keeper) {
            const CounterShard &own = C->shard[blockIdx.x % kShards];
            const float fin = (float)bcast_lane0(load_relaxed(&own.finished));
            const float ac = (float)bcast_lane0(load_relaxed(&own.accepted));
            if (__builtin_amdgcn_readfirstlane(suffice(fin, ac))) return false;
        }
        // lane l reads shard l mod kShards
        const CounterShard *sh = &C->shard[lane & (kShards - 1)];
        unsigned long long va = load_relaxed(&sh->accepted), vf = load_relaxed(&sh->finished);
#pragma unroll
        for (int o = kShards / 2; o > 0; o >>= 1) {
            va += __shfl_xor(va, o, 64);
            vf += __shfl_xor(vf, o, 64);
        }
        const unsigned long long acc = bcast_lane0(va);
        if (acc >= P.target) return false;
        // tiles wanted beyond those taken, by the acceptance of the finished ones
        const float fin = (float)bcast_lane0(vf), ac = (float)acc;
        float est = 4.0f * nx + 256.0f;
        if (acc != 0ull) {
            est = fmaxf((float)P.target * (fin / ac) - nx, 0.0f);
            const bool enough = suffice(fin, ac);
            if (__builtin_amdgcn_readfirstlane(enough && !keeper)) return false;
        }
        rem = fminf(rem, 2.0f * est);
    }
    const int want = (int)fminf(rem * share, (float)kClaimTiles);
    const int len = __builtin_amdgcn_readfirstlane(want < kMinClaim ? kMinClaim : want & ~1);
    b = P.static_tiles +
        bcast_lane0(atomicAdd(&C->next_tile, lane == 0 ? (unsigned long long)len : 0ull));
    e = b + len < P.n_tiles ? b + len : P.n_tiles;
    return b < P.n_tiles;
}

// A workgroup's proposals for the FP64 pass: kept in LDS and passed on with one
// reservation of the list when the workgroup is done, where they fit; otherwise
// one reservation per claim.  The list has one counter, and a reservation waits
// for those before it: a million proposals of which a hundredth is listed took
// 43 us in 4096 reservations of a wave each, K = 8, now 17.
struct DeferList {
    static constexpr unsigned N = 256;
    unsigned long long e[N];
    unsigned n, whole;  // places given out, and those before the first that did not fit
    unsigned long long slot;

    __device__ __forceinline__ void begin()
    {
        if (threadIdx.x == 0) {
            n = 0u;
            whole = N;
        }
    }
    // Lane c holds the bits of tile c of a claim (first proposal i0 + 32 c).
    __device__ __forceinline__ void push(const KernelArgs &a, DevCounters *C, int p, uint64_t i0, uint32_t bits, int lane)
    {
        if (__ballot(bits != 0u) == 0ull) return;
        const int cnt = __popc(bits);
        int incl = cnt;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int up = __shfl_up(incl, o, 64);
            if (lane >= o) incl += up;
        }
        const unsigned total = (unsigned)__builtin_amdgcn_readlane(incl, 63);
        atomicAdd(&C->shard[blockIdx.x % kShards].deferred, lane == 0 ? (unsigned long long)total : 0ull);
        const unsigned at = __builtin_amdgcn_readfirstlane(atomicAdd(&n, lane == 0 ? total : 0u));
        if (at + total <= N && at + total >= at) {
            for (unsigned pos = at + (unsigned)(incl - cnt); bits; bits &= bits - 1, ++pos)
                e[pos] = pack_defer(p, i0 + 32u * lane + (__ffs(bits) - 1));
            return;
        }
        atomicMin(&whole, lane == 0 ? at : N);
        const unsigned long long to = bcast_lane0(atomicAdd(a.defer_count, lane == 0 ? (unsigned long long)total : 0ull));
        for (unsigned long long pos = to + (unsigned)(incl - cnt); bits; bits &= bits - 1, ++pos)
            if (pos < a.defer_cap) a.defer_list[pos] = pack_defer(p, i0 + 32u * lane + (__ffs(bits) - 1));
    }
    // By every thread of the workgroup, its claims done.
    __device__ __forceinline__ void flush(const KernelArgs &a)
    {
        __syncthreads();
        const unsigned m = n < whole ? n : whole;
        if (m == 0u) return;
        if (threadIdx.x == 0) slot = atomicAdd(a.defer_count, (unsigned long long)m);
        __syncthreads();
        for (unsigned i = threadIdx.x; i < m; i += blockDim.x)
            if (slot + i < a.defer_cap) a.defer_list[slot + i] = e[i];
    }
};

__device__ __forceinline__ unsigned int wave_sum_u32(unsigned int v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// What a wave has seen of a point since it last reported: violations of the
// bound and the largest log a.  Reported when the wave leaves the point.
struct PointTally {
    unsigned int n_viol = 0;
    float max_la = -INFINITY;
    __device__ __forceinline__ void report(DevCounters *C, int lane)
    {
        CounterShard &S = C->shard[blockIdx.x % kShards];
        if (__ballot(n_viol != 0u) != 0ull) {
            unsigned int v = n_viol;
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
            add_lane0(&S.violations, v, lane);
        }
        float m = max_la;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o, 64));
        if (__builtin_amdgcn_readfirstlane(__float_as_uint(m)) == __float_as_uint(-INFINITY)) return;  // no work
        const unsigned int key = __builtin_amdgcn_readfirstlane(float_key(m));
        const unsigned int have = __builtin_amdgcn_readfirstlane(
            __hip_atomic_load(&S.max_log_a_key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        if (key > have) atomicMax(&S.max_log_a_key, lane == 0 ? key : 0u);
        n_viol = 0;
        max_la = -INFINITY;
    }
};

// The finished tiles and their definite accepts (lane c: the word of tile c), on
// which claims depend in accepted-count mode.
__device__ __forceinline__ void count_accepted(const DevPoint &P, DevCounters *C, uint32_t word, int len, int lane)
{
    if (P.target == ~0ull) return;
    const unsigned int v = __builtin_amdgcn_readfirstlane(wave_sum_u32(__popc(word)));
    CounterShard &S = C->shard[blockIdx.x % kShards];
    add_lane0(&S.accepted, v, lane);
    add_lane0(&S.finished, (unsigned long long)len, lane);
}

// The waves that stay with point p until its target is met (claim_tiles).
__device__ __forceinline__ bool keeper_wave(int p, unsigned gwave, unsigned W)
{
    return W < 64u || ((gwave + (unsigned)p) & 31u) == 0u;
}

// The work of one wave over the points of a launch: its even share of every
// point, then claims from the points' queues until all are empty.  next()
// gives at most kClaimTiles tiles [base, base + len) of point p.
template <int K>
struct WaveWork {
    unsigned long long cur = 0, end = 0;  // tiles in hand
    int cursor, todo, misses = 0, p = -1; // todo: points whose share has not been taken
    __device__ __forceinline__ WaveWork(unsigned gwave, int n_plist) : cursor((int)(gwave % (unsigned)n_plist)), todo(n_plist) {}
    __device__ __forceinline__ bool next(const KernelArgs &a, const int *plist, int n_plist, unsigned gwave, unsigned W,
                                         float share, int lane, PointTally &tally, unsigned long long &base, int &len)
    {
        // every quantity of this loop is wave-uniform; said for the compiler,
        // which otherwise keeps the point's constants per lane
        while (bcast_lane0(cur) >= bcast_lane0(end)) {
            misses = __builtin_amdgcn_readfirstlane(misses);
            todo = __builtin_amdgcn_readfirstlane(todo);
            cursor = __builtin_amdgcn_readfirstlane(cursor);
            p = __builtin_amdgcn_readfirstlane(p);
            if (misses >= n_plist) {
                if (p >= 0) tally.report(a.cnt + p, lane);
                return false;
            }
            const int q = __builtin_amdgcn_readfirstlane(plist[cursor]);
            if (q != p) {
                if (p >= 0) tally.report(a.cnt + p, lane);
                p = q;
            }
            const DevPoint &P = a.pts[q];
            if (todo > 0) {
                static_range(P, q, gwave, W, cur, end);
                --todo;
                cursor = (cursor + 1 == n_plist) ? 0 : cursor + 1;
            } else if (claim_tiles<K>(P, a.cnt + q, lane, share, keeper_wave(q, gwave, W), cur, end)) {
                misses = 0;
            } else {
                cur = end = 0;
                cursor = (cursor + 1 == n_plist) ? 0 : cursor + 1;
                ++misses;
            }
        }
        base = bcast_lane0(cur);
        const unsigned long long left = bcast_lane0(end) - base;
        len = (int)(left < (unsigned long long)kClaimTiles ? left : (unsigned long long)kClaimTiles);
        cur = base + len;
        return true;
    }
};

// One past the last proposal of a claim of len tiles from base.  The decision
// kernels settle tiles in groups; a claim that is no multiple of the group draws
// the tiles after it and drops them.
__device__ __forceinline__ unsigned long long claim_stop(const DevPoint &P, unsigned long long base, int len)
{
    const unsigned long long e = (base + len) * kTile;
    return e < P.n ? e : P.n;
}

// A lane's share of the statistics of the grid values u = amp u~ of accepted
// samples, from the FP32 values of u~: power sums of u~ in FP64 (scaled by powers
// of amp at the end) and the values above 2 and 4 sigma, counted once per wave.
// Six FP64 operations a value; with the scaling and two counters a lane it took
// twelve instructions where nine do.
struct GridSums {
    double S1 = 0.0, S2 = 0.0, S3 = 0.0, S4 = 0.0;
    unsigned int n_ex = 0, n_ex4 = 0;  // wave-uniform
    float umax = -INFINITY;            // the largest value of this lane's proposal so far

    __device__ __forceinline__ void add(float uf)
    {
        const double u = (double)uf, u2 = u * u;
        S1 += u;
        S2 += u2;
        S3 = __builtin_fma(u2, u, S3);
        S4 = __builtin_fma(u2, u2, S4);
        n_ex += (unsigned)__popcll(__ballot(uf > kTwoSigmaT));  // u > 2 sqrt(E0/pi)
    }
    template <int N>
    __device__ __forceinline__ void add(const float (&uf)[N])
    {
        float top = uf[0];
#pragma unroll
        for (int v = 1; v < N; ++v) top = fmaxf(top, uf[v]);
        umax = fmaxf(umax, top);
        if (__any(top > kFourSigmaT)) {  // u > 4 sqrt(E0/pi): rare
#pragma unroll
            for (int v = 0; v < N; ++v) n_ex4 += (unsigned)__popcll(__ballot(uf[v] > kFourSigmaT));
        }
#pragma unroll
        for (int v = 0; v < N; ++v) {
            add(uf[v]);
            // four values at a time: else the masks of all N wait in SGPRs
            if (v % 4 == 3) {
                n_ex = __builtin_amdgcn_readfirstlane(n_ex);
                asm volatile("" : "+s"(n_ex), "+v"(S1), "+v"(S2), "+v"(S3), "+v"(S4));
            }
        }
    }
};

// First piece of point p (p = n_points: their number), and log2 of its pieces' length.
__device__ __forceinline__ unsigned long long cut_first(const Cuts *c, int p)
{
    return c->at[p] & ((1ull << kCutShiftBit) - 1);
}
__device__ __forceinline__ int cut_shift(const Cuts *c, int p) { return (int)(c->at[p] >> kCutShiftBit); }

// The point of piece i, by a wave: 64 points looked at together.
__device__ __forceinline__ int point_of_cut(const Cuts *c, int n_points, unsigned long long i, int lane)
{
    int lo = 0, n = n_points;
    while (n > 1) {
        const int step = (n + kWave - 1) / kWave;
        const unsigned long long first = step * lane < n ? cut_first(c, lo + step * lane) : ~0ull;
        const int q = __popcll(__ballot(first <= i)) - 1;  // the one at lo begins there or before
        lo += step * q;
        n = n - step * q < step ? n - step * q : step;
    }
    return lo;
}

// Exclusive prefix of v over a workgroup of B threads, and the sum of all.
template <int B>
__device__ __forceinline__ unsigned long long block_prefix(unsigned long long v, unsigned long long (&wsum)[B / kWave],
                                                           unsigned long long &all)
{
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    unsigned long long incl = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const unsigned long long up = __shfl_up(incl, o, 64);
        if (lane >= o) incl += up;
    }
    __syncthreads();  // wsum of the last call has been read
    if (lane == 63) wsum[wv] = incl;
    __syncthreads();
    unsigned long long before = 0;
    all = 0;
    for (int w = 0; w < B / kWave; ++w) {
        before += w < wv ? wsum[w] : 0ull;
        all += wsum[w];
    }
    return before + incl - v;
}

// Fills c from every point's number of pieces and their log2 length, piece(p, sh)
// (one workgroup of B threads).
template <int B, class Piece>
__device__ void place_cuts(Cuts *c, int n_points, Piece piece)
{
    __shared__ unsigned long long wsum[B / kWave];
    const int tid = threadIdx.x;
    unsigned long long run = 0;
    for (int p0 = 0; p0 < n_points; p0 += B) {
        const int p = p0 + tid;
        int sh = 0;
        const unsigned long long v = p < n_points ? piece(p, sh) : 0ull;
        unsigned long long all;
        const unsigned long long before = run + block_prefix<B>(v, wsum, all);
        if (p < n_points) c->at[p] = before | ((unsigned long long)sh << kCutShiftBit);
        run += all;
    }
    if (tid == 0) c->at[n_points] = run;
}

// The segments of a call from the tiles decided (one workgroup of B threads).
template <int B>
__device__ void plan_segments(const KernelArgs &a)
{
    __shared__ unsigned long long words[B];
    const int tid = threadIdx.x;
    unsigned long long sum = 0;
    for (int p = tid; p < a.n_points; p += B) sum += tiles_taken(a.pts[p], a.cnt[p].next_tile);
    words[tid] = sum;
    __syncthreads();
    for (int o = B / 2; o > 0; o >>= 1) {
        if (tid < o) words[tid] += words[tid + o];
        __syncthreads();
    }
    const int shift = seg_shift_for(words[0]);
    place_cuts<B>(a.seg, a.n_points, [&](int p, int &sh) {
        sh = shift;
        return (tiles_taken(a.pts[p], a.cnt[p].next_tile) + (1ull << shift) - 1) >> shift;
    });
}

__device__ __forceinline__ unsigned long long read_lane_u64(unsigned long long v, int l)
{
    const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)v, l);
    const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(v >> 32), l);
    return ((unsigned long long)hi << 32) | lo;
}

// Inclusive prefix sum over the wave's lanes (all of them active), in registers.
__device__ __forceinline__ int wave_prefix_i32(int v)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);  // row_shr 1, 2, 4, 8: within 16 lanes
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);  // lane 15 of a row to the next: rows 1 and 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);  // lane 31 to rows 2 and 3
    return v;
}

// The accepted proposals of ranks [first, end) of a point, in order, for one wave:
// from the segment on that holds the first of them it reads the accept words in
// groups of GW (one per lane), kAhead groups at a time, and queues the offsets of
// their accepted proposals in LDS; the part of a tile of TILE that is left waits in
// registers.
template <int GW, int TILE>
struct RankReader {
    static_assert(GW <= kWave && kWave % TILE == 0, "a word per lane, and a waiting proposal");
    // groups loaded together: where few are accepted the loads are what a group takes (4096
    // samples among 3e6 words at K = 32: 0.4 ms more, one at a time); twice as many are no faster
    static constexpr int kAhead = GW / 4;
    static constexpr int N = GW * 32;  // offsets queued at a time: any group's
    static_assert(kAhead * N <= 1 << 16, "offsets of 16 bits");
    uint16_t *list;                    // N of LDS, this wave's
    const uint32_t *words;
    const PointRanks &R;
    const unsigned long long *seg_base;  // KernelArgs
    int shift;                           // log2 of a segment's words
    unsigned long long n_words, at = 0, after = 0;  // the point's accept words; the first of those queued, and after them
    unsigned long long rank, end;        // rank of the first proposal not done yet
    unsigned long long held = 0;         // the proposal that waits at place lane % TILE
    int n_held = 0, fresh = 0;           // how many wait; how many are queued
    int skip;                            // accepted ones still to pass before the first

    __device__ __forceinline__ RankReader(const KernelArgs &a, const PointRanks &R_, unsigned long long bm_off, uint16_t *lds,
                                          unsigned long long first_, unsigned long long end_, int lane)
        : list(lds), words(a.bitmap + bm_off), R(R_), seg_base(a.seg_base),
          shift(__builtin_amdgcn_readfirstlane(R_.seg_shift)), n_words(bcast_lane0(R_.n_words)),
          rank(bcast_lane0(first_)), end(bcast_lane0(end_))
    {
        skip = (int)(rank - seek(rank, 0ull, lane));
    }
    // To the segment that holds rank r, the last that begins there or before, if that is
    // ahead: it is looked for in 64 segments together, from `from` on; the rank it
    // begins at.
    __device__ __forceinline__ unsigned long long seek(unsigned long long r, unsigned long long from, int lane)
    {
        const unsigned long long *base0 = seg_base + bcast_lane0(R.seg_first), before0 = bcast_lane0(R.base);
        unsigned long long lo = from, n = bcast_lane0(R.n_segs) - from, before = 0;
        while (n > 1) {
            const unsigned long long step = (n + kWave - 1) / kWave, i = step * lane;
            const unsigned long long base = i < n ? base0[lo + i] - before0 : ~0ull;
            const int c = __popcll(__ballot(base <= r)) - 1;  // the one at lo begins there or before
            before = read_lane_u64(base, c);
            lo += step * c;
            n = n - step * c < step ? n - step * c : step;
        }
        at = at > lo << shift ? at : lo << shift;
        return before;
    }
    // From word `from` on nothing was found before `at`: if that is another segment, past
    // those that hold none before rank r.
    __device__ __forceinline__ void skip_empty(unsigned long long r, unsigned long long from, int lane)
    {
        if (at >> shift == from >> shift || at >= n_words) return;
        const unsigned long long cur = at >> shift, i = cur + lane;
        const unsigned long long base = i < R.n_segs ? seg_base[R.seg_first + i] - R.base : ~0ull;
        const int c = __popcll(__ballot(base <= r)) - 1;
        if (c == kWave - 1) seek(r, cur + c, lane);
        else if (c > 0) at = (cur + c) << shift;
    }
    // Queues the next proposals: how many, with those that wait, a multiple of TILE or
    // all that are left, or 0 when all are done.
    __device__ __forceinline__ int next(int lane)
    {
        while (rank < end && at < n_words) {
            uint32_t ahead[kAhead], some = 0u;  // some: the groups that hold any
#pragma unroll
            for (int h = 0; h < kAhead; ++h) {
                const unsigned long long w = at + h * GW + lane;
                ahead[h] = lane < GW && w < n_words ? words[w] : 0u;
            }
#pragma unroll
            for (int h = 0; h < kAhead; ++h) some |= __ballot(ahead[h] != 0u) != 0ull ? 1u << h : 0u;
            const bool none = some == 0u;
            const unsigned long long want = end - rank - n_held;
            bool last = false;
            fresh = 0;
            after = at + kAhead * GW;
            for (; some; some &= some - 1) {
                const int h0 = __ffs(some) - 1;
                uint32_t word = ahead[0];
#pragma unroll
                for (int h = 1; h < kAhead; ++h) word = h0 == h ? ahead[h] : word;
                const int cntw = __popc(word);
                const int incl = wave_prefix_i32(cntw);
                const int total = __builtin_amdgcn_readlane(incl, 63);
                if (total <= skip) {
                    skip -= total;
                    continue;
                }
                if (fresh + total - skip > N) {  // no room: the next time
                    after = at + h0 * GW;
                    break;
                }
                int pos = fresh + incl - cntw - skip;
                for (uint32_t m = word; m; m &= m - 1, ++pos)
                    if (pos >= fresh) list[pos] = (uint16_t)((h0 * GW + lane) * 32 + __ffs(m) - 1);
                fresh += total - skip;
                skip = 0;
                last = (unsigned long long)fresh >= want;
                if (last) break;
            }
            wave_lds_sync();
            if (last) {
                fresh = (int)want;
                return n_held + fresh;
            }
            if (n_held + fresh >= TILE) return (n_held + fresh) & ~(TILE - 1);
            keep(0, lane);
            const unsigned long long from = at;
            at = after;
            if (none) skip_empty(rank + n_held, from, lane);
        }
        return 0;
    }
    // The e-th of them (e = lane modulo TILE), from the point's first proposal.
    __device__ __forceinline__ unsigned long long local(int e) const
    {
        return e < n_held ? held : at * kTile + list[e - n_held];
    }
    // n of them are done (what next gave).
    __device__ __forceinline__ void done(int n, int lane)
    {
        rank += n;
        keep(n, lane);
        at = after;
    }
    // All but the first n wait, fewer than TILE.
    __device__ __forceinline__ void keep(int n, int lane)
    {
        const int left = n_held + fresh - n, q = lane % TILE;
        if (n == 0 ? q >= n_held && q < left : q < left) held = at * kTile + list[n + q - n_held];
        n_held = left;
        wave_lds_sync();
    }
};

// Per-wave u(0) histogram in LDS, kept while the wave stays with one point and
// added to the point's global one (a shard per workgroup) when it leaves.
struct WaveHist {
    unsigned int *bins;  // this wave's kNBins counters
    int p = -1;
    __device__ __forceinline__ void enter(const KernelArgs &a, int q, int lane)
    {
        if (q == p) return;
        flush(a, lane);
        bins[lane] = 0u;
        p = q;
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
    __device__ __forceinline__ void flush(const KernelArgs &a, int lane)
    {
        if (p < 0) return;
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
        const unsigned int c = bins[lane];
        if (c) atomicAdd(&a.hist[((size_t)p * kShards + blockIdx.x % kShards) * kNBins + lane], (unsigned long long)c);
    }
};
static_assert(kNBins == kWave, "one bin per lane");


__device__ __forceinline__ double wave_sum_f64(double v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// log f = -beta'/(E0 K^2) (H2 - c H3) in FP64 at a point x of the sphere with
// t = sum k^2 s_k: H2 = E0 t by Parseval and H3 by the double sum over the
// triads k + (n - k) = n (Sec. IV.A).
__device__ inline double log_f_fp64(int K, double E0, double beta_p, double c32, const double *x, double t)
{
    const double pi = 3.14159265358979323846;
    const double s = sqrt(E0 / (2.0 * pi));
    double tri = 0.0;
    for (int n = 2; n <= K; ++n) {
        double in_re = 0.0, in_im = 0.0;
        for (int k = 1; k < n; ++k) {
            const double pr = s * x[k - 1], pi_ = -s * x[K + k - 1];
            const double qr = s * x[n - k - 1], qi = -s * x[K + n - k - 1];
            in_re += pr * qr - pi_ * qi;
            in_im += pr * qi + pi_ * qr;
        }
        tri += (s * x[n - 1]) * in_re + (-s * x[K + n - 1]) * in_im;
    }
    const double H3 = 2.0 * pi * tri;
    const double H2 = E0 * t;
    return -(beta_p / (E0 * (double)K * K) * (H2 - c32 * H3));
}

// ---------------------------------------------------------------------------
// Learned mixture proposal
// ---------------------------------------------------------------------------
// Component of a proposal from its component word: -1 (g_Sigma) when w < E,
// else j = (w - E) div B, formed in integers (one FP32 estimate, corrected
// by one step: the estimate is within 1 of the quotient).
__device__ __forceinline__ int mix_component(const DevMix &M, uint32_t w)
{
    const uint32_t d = w - M.E;
    uint32_t j = (uint32_t)((float)d * M.invB);
    j = j > (uint32_t)(kMixS - 1) ? (uint32_t)(kMixS - 1) : j;
    const uint32_t prod = j * M.B;
    if (prod > d) --j;
    else if (d - prod >= M.B) ++j;
    return w < M.E ? -1 : (int)j;
}

// Draw of proposal i from q_mix: this lane's K coordinates of X (words
// 0..2K-1 as for the paper's proposal, 2K+1 the component word, 2K+2 and 2K+3
// the pair eta; wl is the last Philox block) and its parts of |X|^2, of
// sum_k k^2 X_k^2 and of Qa = sum a_c X_c^2.  rv points to the RV table of the
// point (LDS or global memory).  FAST as for gen_x_part.
template <int K, bool FAST>
__device__ __forceinline__ void gen_x_mix_part(const DevPoint &P, const DevMix &M, const float *rv, uint64_t i, int half,
                                               float (&x)[K], float &r2, float &tk, float &qa)
{
    const uint32_t c0 = (uint32_t)i, c1 = (uint32_t)(i >> 32), c2 = P.point_id;
    draw_blocks<K / 4, FAST>(c0, c1, c2, (uint32_t)(half * (K / 4)), P.key0, P.key1, x);
    const uint4 wl = philox4x32_10(c0, c1, c2, (uint32_t)(K / 2), P.key0, P.key1);
    const int comp = mix_component(M, wl.y);
    const bool def = comp < 0;
    float eta[2];
    if constexpr (FAST) {
        const uint32_t w1[1] = {wl.z}, w2[1] = {wl.w};
        draw_fast<1>(w1, w2, eta);
    } else {
        box_muller_f32(wl.z, wl.w, eta[0], eta[1]);
    }
    const float e0 = def ? 0.0f : eta[0], e1 = def ? 0.0f : eta[1];
    const float2 *row = reinterpret_cast<const float2 *>(rv + (2 * (def ? 0 : comp) + half) * (2 * K + 2));
#pragma unroll
    for (int j = 0; j < K; ++j) {
        const float sc = def ? P.sig[j] : M.sqd[j];
        const float2 v = row[j];
        x[j] = __builtin_fmaf(v.x, e0, __builtin_fmaf(v.y, e1, sc * x[j]));
        if (j % 8 == 7) __builtin_amdgcn_sched_barrier(0);  // the loads of eight coordinates at a time
    }
    r2 = tk = qa = 0.0f;
    const ConstFloats am = const_floats(M.a);
#pragma unroll
    for (int j = 0; j < K; ++j) {
        const float sq = x[j] * x[j];
        r2 += sq;
        tk = __builtin_fmaf((float)((j + 1) * (j + 1)), sq, tk);
        qa = __builtin_fmaf(am[j], sq, qa);
    }
}

// The projected point of proposal i of the mixture sampler (rows for the caller).
template <int K>
__device__ __forceinline__ void gen_xhat_mix(const DevPoint &P, const DevMix &M, const float *rv, uint64_t i, int half,
                                             float (&x)[K], float &t)
{
    float r2, tk, qa;
    gen_x_mix_part<K, false>(P, M, rv, i, half, x, r2, tk, qa);
    const float inv = __builtin_amdgcn_rsqf(sum32(r2));
    t = sum32(tk) * (inv * inv);
#pragma unroll
    for (int j = 0; j < K; ++j) x[j] *= inv;
}

// z = (R_j A V C^T)^T X for the S shifts on the matrix cores (C^T C = G^-1, so
// that y_j^T G^-1 y_j = |z_j|^2): row tile q holds rank index q, row j the
// shift, column the proposal (the B operand layout).  Row tiles share their row
// order, so y0[v] and y1[v] are the two entries of one shift's z.
template <int K, int PREC>
__device__ __forceinline__ void mix_y(const float (&x)[K], const bf16x8 (&bh)[K / 8], const bf16x8 (&bl)[K / 8],
                                      const char *yt_hi, const char *yt_lo, int lane, f32x16 &y0, f32x16 &y1)
{
    if constexpr (PREC == PREC_FP32) {
        const float4 *tab = reinterpret_cast<const float4 *>(yt_hi);
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            f32x16 acc = {};
#pragma unroll
            for (int q = 0; q < K / 4; ++q) {
                float4 a = tab[(t * (K / 4) + q) * kWave + lane];
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.x, x[4 * q + 0], acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.y, x[4 * q + 1], acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.z, x[4 * q + 2], acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.w, x[4 * q + 3], acc, 0, 0, 0);
            }
            if (t == 0) y0 = acc; else y1 = acc;
        }
    } else {
        const bf16x8 *th = reinterpret_cast<const bf16x8 *>(yt_hi);
        const bf16x8 *tl = reinterpret_cast<const bf16x8 *>(yt_lo);
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            f32x16 acc = {};
#pragma unroll
            for (int s = 0; s < K / 8; ++s) {
                const int idx = (t * (K / 8) + s) * kWave + lane;
                const bf16x8 ah = th[idx];
                if constexpr (PREC == PREC_BF16X3) {
                    const bf16x8 al = tl[idx];
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al, bh[s], acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bl[s], acc, 0, 0, 0);
                }
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bh[s], acc, 0, 0, 0);
            }
            if (t == 0) y0 = acc; else y1 = acc;
        }
    }
}

// The same products from the parity-split operands (split_eo) against the
// y tables staged in the parity layout (stage_parity_frags, 2 row tiles); the
// two row tiles accumulate as independent chains.  FP32 reads x as mix_y.
template <int K, int PREC>
__device__ __forceinline__ void mix_y_eo(const float (&x)[K], const bf16x8 (&eh)[K / 16], const bf16x8 *el,
                                         const bf16x8 (&oh)[K / 16], const bf16x8 *ol, const char *yt_hi,
                                         const char *yt_lo, int lane, f32x16 &y0, f32x16 &y1)
{
    if constexpr (PREC == PREC_FP32) {
        bf16x8 bh[K / 8], bl[K / 8];
        mix_y<K, PREC>(x, bh, bl, yt_hi, yt_lo, lane, y0, y1);
    } else {
        constexpr int S = eo_steps<K>();
        const bf16x8 *th = reinterpret_cast<const bf16x8 *>(yt_hi);
        const bf16x8 *tl = reinterpret_cast<const bf16x8 *>(yt_lo);
        f32x16 acc[2] = {f32x16{}, f32x16{}};
#pragma unroll
        for (int s = 0; s < S; ++s)
#pragma unroll
            for (int p = 0; p < 2; ++p)
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    const int idx = ((t * S + s) * 2 + p) * kWave + lane;
                    const bf16x8 &bh = p == 0 ? eh[s] : oh[s];
                    const bf16x8 ah = th[idx];
                    if constexpr (PREC == PREC_BF16X3) {
                        const bf16x8 &bl = p == 0 ? el[s] : ol[s];
                        const bf16x8 al = tl[idx];
                        acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al, bh, acc[t], 0, 0, 0);
                        acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bl, acc[t], 0, 0, 0);
                    }
                    acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bh, acc[t], 0, 0, 0);
                }
        y0 = acc[0];
        y1 = acc[1];
    }
}

// log q_mix in FP32 from the shifts' z, Qa = X^T A X (both unprojected: the
// ratios r_j = qf_j/Q = 1 - |z_j|^2/Qa are scale free), |X|^-2 and t.
//   ln q_net + ln(1 - eps) = c_net - K ln(Qa |X|^-2) + ln sum_j r_j^-K,
//   ln(eps g_Sigma) = c_g - K ln(1 + alpha beta' t/K^3).
// The sum is taken relative to the smallest r_j of the proposal (all terms
// <= 1, the largest exactly 1).  mix_shift_sum: this lane's 16 terms, and
// log2 of the smallest ratio over both lanes; mix_log_q_f32: the rest, from the
// sum over both lanes.
__device__ __forceinline__ float mix_shift_sum(const f32x16 &y0, const f32x16 &y1, float Qa, float Kf, float &lmin)
{
    const float invQ = __builtin_amdgcn_rcpf(Qa);
    float l[16];
    lmin = INFINITY;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const float a0 = y0[v], a1 = y1[v];
        const float quad = __builtin_fmaf(a0, a0, a1 * a1);
        const float r = fmaxf(__builtin_fmaf(-quad, invQ, 1.0f), 1e-30f);
        l[v] = log2_hw(r);
        lmin = fminf(lmin, l[v]);
    }
    float lo = lmin, hi = lmin;
    swap32(lo, hi);
    lmin = fminf(lo, hi);
    // K (lmin - l) as one FMA: K is a power of two (8, 16, 32), so K lmin is
    // exact and the FMA rounds the same exact value as the difference scaled
    const float klmin = Kf * lmin;
    float sum = __builtin_amdgcn_exp2f(__builtin_fmaf(-Kf, l[0], klmin));
#pragma unroll
    for (int v = 1; v < 16; ++v) sum += __builtin_amdgcn_exp2f(__builtin_fmaf(-Kf, l[v], klmin));
    return sum;
}
__device__ __forceinline__ float mix_log_q_f32(const DevPoint &P, const DevMix &M, float sum, float lmin, float Qa,
                                               float inv2, float t, float Kf)
{
    const float ln2 = 0.69314718055994531f;
    const float LN = M.c_net + ln2 * (log2_hw(sum) - Kf * (lmin + log2_hw(Qa * inv2)));
    const float LG = M.c_g - Kf * log1p_f32(P.g_coef * t);
    const float hi = fmaxf(LN, LG);
    return hi + log1p_f32(__builtin_amdgcn_exp2f(-fabsf(LN - LG) * 1.4426950408889634f));
}

}  // namespace tkdv
