// Extreme wave fields among stored samples (Sec. V, the search of individual
// samples for the largest surface displacement):
//   k_grid_max   per row x^: u on the N = 4K grid (u = amp Phi^T x^, FP32
//                matrix products from the FP32 synthesis tables in LDS), its
//                maximum, the first grid index attaining it, and the count of
//                rows whose maximum exceeds a threshold (K <= 32);
//   k_grid_max_q the same in the quarter-period form (K = 64, 128);
// Both count the maxima's order-preserving keys by their top 8 bits.  Then an
// exact radix select with no step on the host:
//   k_key_hist   takes the next 8 bits of the selected key from the last counts
//                and counts the keys that share it by the bits after;
//   k_key_collect takes the last 8 bits and lists the rows above the selected
//                key and the rows equal to it.
#include "tkdv_device.h"
#include "tkdv_extremes.h"
#include "tkdv_internal.h"

namespace tkdv {
namespace {

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

// Order-preserving map float -> uint32 (larger float, larger key).
__device__ __forceinline__ uint32_t max_key(float f)
{
    const uint32_t u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Keys of one workgroup by 8 bits, added to its shard of the call's counts.
__device__ __forceinline__ void flush_hist(const uint32_t *h, unsigned long long *hist)
{
    __syncthreads();
    for (int b = threadIdx.x; b < kExtBins; b += blockDim.x)
        if (h[b]) atomicAdd(&hist[(blockIdx.x % kExtShards) * kExtBins + b], (unsigned long long)h[b]);
}

// Bound by the FP32 products; the next tile's rows are loaded beside them.
template <int K>
__global__ void __launch_bounds__(kExtBlock) k_grid_max(ExtArgs a)
{
    extern __shared__ __attribute__((aligned(16))) char lds[];
    __shared__ uint32_t h[kExtBins];
    if (threadIdx.x < kExtBins) h[threadIdx.x] = 0u;
    constexpr int T = K / 8, Q = K / 4;
    constexpr int tab = T * Q * kWave * 16;  // FP32 table bytes
    {
        const uint4 *s0 = reinterpret_cast<const uint4 *>(a.phi_f32);
        uint4 *d = reinterpret_cast<uint4 *>(lds);
        for (int v = threadIdx.x; v < tab / 16; v += kExtBlock) d[v] = s0[v];
    }
    __syncthreads();
    const float4 *tb = reinterpret_cast<const float4 *>(lds);
    const int lane = threadIdx.x & 63, half = lane >> 5, pl = lane & 31;
    const unsigned long long n_tiles = (a.n + kTile - 1) / kTile;
    const unsigned long long waves = (unsigned long long)gridDim.x * (kExtBlock / kWave);
    unsigned long long n_exc = 0;
    float4 next[Q];
    auto load = [&](unsigned long long tile) {
        const unsigned long long row = tile * kTile + pl;
        const float4 *src = reinterpret_cast<const float4 *>(a.xhat + (row < a.n ? row : 0ull) * a.stride + half * K);
#pragma unroll
        for (int q = 0; q < Q; ++q) next[q] = src[q];
    };
    const unsigned long long tile0 =
        __builtin_amdgcn_readfirstlane(blockIdx.x * (kExtBlock / kWave) + (threadIdx.x >> 6));
    if (tile0 < n_tiles) load(tile0);
    for (unsigned long long tile = tile0; tile < n_tiles; tile += waves) {
        const unsigned long long row = tile * kTile + pl;
        const bool valid = row < a.n;
        float x[K];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const float4 v = next[q];
            x[4 * q + 0] = v.x;
            x[4 * q + 1] = v.y;
            x[4 * q + 2] = v.z;
            x[4 * q + 3] = v.w;
        }
        if (tile + waves < n_tiles) load(tile + waves);
        float best = -INFINITY;
        int bj = 0;
        constexpr int kTileUnroll = T < 4 ? T : 2;  // grid tiles unrolled
#pragma unroll kTileUnroll
        for (int t = 0; t < T; ++t) {
            f32x16 acc = {};
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const float4 c = tb[(t * Q + q) * kWave + lane];
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(c.x, x[4 * q + 0], acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(c.y, x[4 * q + 1], acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(c.z, x[4 * q + 2], acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(c.w, x[4 * q + 3], acc, 0, 0, 0);
            }
            // acc[v] of lane l: grid point 32 t + 8 (v/4) + 4 (l/32) + v%4 of row l%32;
            // v increases with the grid index within each half
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int j = 32 * t + 8 * (v >> 2) + 4 * half + (v & 3);
                if (acc[v] > best) {
                    best = acc[v];
                    bj = j;
                }
            }
        }
        // the other half of the row: larger value, or the lower index on a tie
        const float ob = __shfl_xor(best, 32, 64);
        const int oj = __shfl_xor(bj, 32, 64);
        if (ob > best || (ob == best && oj < bj)) {
            best = ob;
            bj = oj;
        }
        const float um = best * a.amp;
        const bool exc = valid && half == 0 && um > a.threshold;
        n_exc += __popcll(__ballot(exc));
        if (valid && half == 0) {
            const uint32_t key = max_key(um);
            a.keys[row] = key;
            atomicAdd(&h[key >> 24], 1u);
            if (a.umax) a.umax[row] = um;
            if (a.jmax) a.jmax[row] = bj;
        }
    }
    // n_exc is the same in every lane (sums of ballots)
    const unsigned long long tot = ((unsigned long long)__builtin_amdgcn_readfirstlane((uint32_t)(n_exc >> 32)) << 32) |
                                   __builtin_amdgcn_readfirstlane((uint32_t)n_exc);
    if (tot) atomicAdd(a.n_exceed, lane == 0 ? tot : 0ull);
    flush_hist(h, a.hist);
}

// K = 64 and 128: the quarter-period form of the same grid maximum, on the
// grid xi_j = -pi + 2 pi j/N itself.  Representatives xi_rho = 2 pi rho/N,
// rho < K, from the FP32 statistics tables in LDS (16 rho per tile, outputs
// Ce, Co, Se, So: the cos/sin sums over even/odd modes); each gives u at
// xi (grid index 2K + rho), xi - pi (rho), -xi (2K - rho) and pi - xi
// (4K - rho), rho = 0 only the first two; +-pi/2 (3K and K) come from direct
// sums.  A quarter of the dense form's products.  A wave takes 16 rows at a
// time: lane l holds coordinates [K/4 (l/16), K/4 (l/16 + 1)) of both blocks
// of row l % 16 (the B operand of the 16x16x4 products, mode index on l/16).
template <int K>
struct ExtQ {
    static constexpr int CPL = K / 4, TILES = K / 16, QG = K / 32;
    static constexpr int TAB_BYTES = TILES * 4 * QG * kWave * 16;
    static constexpr int BLOCK = 512;
};

// Four running maxima a lane, one for each of the four points of a
// representative: their grid indices rise or fall with rho, so that a tie is
// settled by > or >= alone (three instructions a value instead of seven; rho = 0
// enters twice with the same values).  Where a row's maximum is -inf (values of
// -inf and NaN only) no index has been kept and the row's tile is taken again
// with every index compared.  Bound by reading the rows (512 bytes each at K = 64)
// with the products beside it, hence the next rows loaded ahead: 1e6 rows at
// K = 64, 230 us, now 190.
template <int K>
__global__ void __launch_bounds__(ExtQ<K>::BLOCK) k_grid_max_q(ExtArgs a)
{
    constexpr int CPL = ExtQ<K>::CPL, QG = ExtQ<K>::QG, B = ExtQ<K>::BLOCK, NV = CPL / 4;
    extern __shared__ __attribute__((aligned(16))) char lds[];
    __shared__ uint32_t h[kExtBins];
    if (threadIdx.x < kExtBins) h[threadIdx.x] = 0u;
    {
        const uint4 *s0 = reinterpret_cast<const uint4 *>(a.phi_f32);
        uint4 *d = reinterpret_cast<uint4 *>(lds);
        for (int v = threadIdx.x; v < ExtQ<K>::TAB_BYTES / 16; v += B) d[v] = s0[v];
    }
    __syncthreads();
    const float4 *tab = reinterpret_cast<const float4 *>(lds);
    const int lane = threadIdx.x & 63, g = lane >> 4, pl = lane & 15;
    const unsigned long long n_chunks = (a.n + 15) / 16;
    const unsigned long long waves = (unsigned long long)gridDim.x * (B / kWave);
    unsigned long long n_exc = 0;
    float4 next[2 * NV];
    auto load = [&](unsigned long long ch) {
        const unsigned long long row = ch * 16 + pl;
        const float4 *src = reinterpret_cast<const float4 *>(a.xhat + (row < a.n ? row : 0ull) * a.stride + CPL * g);
#pragma unroll
        for (int q = 0; q < NV; ++q) {
            next[q] = src[q];
            next[NV + q] = src[K / 4 + q];
        }
    };
    const unsigned long long ch0 = __builtin_amdgcn_readfirstlane(blockIdx.x * (B / kWave) + (threadIdx.x >> 6));
    if (ch0 < n_chunks) load(ch0);
    for (unsigned long long ch = ch0; ch < n_chunks; ch += waves) {
        const unsigned long long row = ch * 16 + pl;
        const bool valid = row < a.n;
        float c[CPL], s[CPL];
#pragma unroll
        for (int q = 0; q < NV; ++q) {
            const float4 vc = next[q], vs = next[NV + q];
            c[4 * q + 0] = vc.x;
            c[4 * q + 1] = vc.y;
            c[4 * q + 2] = vc.z;
            c[4 * q + 3] = vc.w;
            s[4 * q + 0] = vs.x;
            s[4 * q + 1] = vs.y;
            s[4 * q + 2] = vs.z;
            s[4 * q + 3] = vs.w;
        }
        if (ch + waves < n_chunks) load(ch + waves);
        float best = -INFINITY;
        int bj = 0x7fffffff;
        auto take = [&](float u, int j) {
            if (u > best || (u == best && j < bj)) {
                best = u;
                bj = j;
            }
        };
        // the grid values of the representatives, to use(points, code = 4 tau + v)
        auto grid_values = [&](auto use) {
#pragma unroll 1
            for (int tau = 0; tau < ExtQ<K>::TILES; ++tau) {
                f32x4 acc[4] = {f32x4{}, f32x4{}, f32x4{}, f32x4{}};
#pragma unroll
                for (int q4 = 0; q4 < QG; ++q4)
#pragma unroll
                    for (int o = 0; o < 4; ++o) {
                        // out o: 0 Ce, 1 Co, 2 Se, 3 So; mode K/4 g + 2 idx + 2 (even) or + 1 (odd)
                        const float4 av = tab[((tau * 4 + o) * QG + q4) * kWave + lane];
                        const float *v = (o < 2) ? c : s;
                        const int par = (o == 0 || o == 2) ? 1 : 0;
                        acc[o] = __builtin_amdgcn_mfma_f32_16x16x4f32(av.x, v[2 * (4 * q4 + 0) + par], acc[o], 0, 0, 0);
                        acc[o] = __builtin_amdgcn_mfma_f32_16x16x4f32(av.y, v[2 * (4 * q4 + 1) + par], acc[o], 0, 0, 0);
                        acc[o] = __builtin_amdgcn_mfma_f32_16x16x4f32(av.z, v[2 * (4 * q4 + 2) + par], acc[o], 0, 0, 0);
                        acc[o] = __builtin_amdgcn_mfma_f32_16x16x4f32(av.w, v[2 * (4 * q4 + 3) + par], acc[o], 0, 0, 0);
                    }
#pragma unroll
                for (int v = 0; v < 4; ++v) {  // acc[o][v] of lane l: representative rho = 16 tau + 4 (l/16) + v
                    const float pe = acc[0][v] + acc[1][v], me = acc[0][v] - acc[1][v];
                    const float ps = acc[2][v] + acc[3][v], ms = acc[2][v] - acc[3][v];
                    const float u[4] = {me + ms, pe - ps, pe + ps, me - ms};  // xi - pi, -xi, xi, pi - xi
                    use(u, 4 * tau + v);
                }
            }
        };
        auto rho_of = [&](int code) { return 16 * (code >> 2) + 4 * g + (code & 3); };
        // grid index of point o of representative rho: rises with rho (o = 0, 2) or falls
        auto index_of = [&](int o, int rho) {
            return o == 0 ? rho : (o == 1 ? 2 * K - rho : (o == 2 ? 2 * K + rho : 4 * K - rho));
        };
        float ub[4] = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
        int uc[4] = {-1, -1, -1, -1};
        grid_values([&](const float (&u)[4], int code) {
#pragma unroll
            for (int o = 0; o < 4; ++o) {
                const bool up = (o & 1) ? u[o] >= ub[o] : u[o] > ub[o];
                ub[o] = up ? u[o] : ub[o];
                uc[o] = up ? code : uc[o];
            }
        });
#pragma unroll
        for (int o = 0; o < 4; ++o)
            if (uc[o] >= 0) take(ub[o], index_of(o, rho_of(uc[o])));
        // xi = +-pi/2: mode K g/4 + j + 1 is j + 1 modulo 4
        float Av = 0.0f, Bv = 0.0f;
#pragma unroll
        for (int j = 0; j < CPL; j += 4) {
            Av += c[j + 3] - c[j + 1];
            Bv += s[j] - s[j + 2];
        }
        Av += __shfl_xor(Av, 16, 64);
        Av += __shfl_xor(Av, 32, 64);
        Bv += __shfl_xor(Bv, 16, 64);
        Bv += __shfl_xor(Bv, 32, 64);
        if (g == 0) {
            take(Av + Bv, 3 * K);  // pi/2
            take(Av - Bv, K);      // -pi/2
        }
        // the row's grid values are split over lanes l, l ^ 16, l ^ 32, l ^ 48
        auto merge = [&]() {
#pragma unroll
            for (int m = 16; m <= 32; m <<= 1) {
                const float ob = __shfl_xor(best, m, 64);
                const int oj = __shfl_xor(bj, m, 64);
                take(ob, oj);
            }
        };
        merge();
        if (__any(best == -INFINITY)) {
            grid_values([&](const float (&u)[4], int code) {
                const int rho = rho_of(code);
#pragma unroll
                for (int o = 0; o < 4; ++o)
                    if (!(o & 1) || rho != 0) take(u[o], index_of(o, rho));
            });
            merge();
        }
        if (bj == 0x7fffffff) bj = 0;  // no value compared (a row of NaN)
        const float um = best * a.amp;
        const bool exc = valid && g == 0 && um > a.threshold;
        n_exc += __popcll(__ballot(exc));
        if (valid && g == 0) {
            const uint32_t key = max_key(um);
            a.keys[row] = key;
            atomicAdd(&h[key >> 24], 1u);
            if (a.umax) a.umax[row] = um;
            if (a.jmax) a.jmax[row] = bj;
        }
    }
    if (lane == 0 && n_exc) atomicAdd(a.n_exceed, n_exc);
    flush_hist(h, a.hist);
}

// The digit of the need-th largest key by the counts of one level (a workgroup
// of kExtSelBlock threads): the largest with at least need keys at or above it;
// need becomes what is left of it.
__device__ uint32_t select_digit(const unsigned long long *hist, unsigned long long &need)
{
    __shared__ unsigned long long at[kExtBins + 1];  // keys of digit b and above
    __shared__ uint32_t digit_s;
    const int b = threadIdx.x;
    if (b < kExtBins) {
        unsigned long long v = 0;
        for (int s = 0; s < kExtShards; ++s) v += hist[s * kExtBins + b];
        at[b] = v;
    }
    if (b == 0) {
        at[kExtBins] = 0;
        digit_s = 0u;
    }
    __syncthreads();
    for (int o = 1; o < kExtBins; o <<= 1) {
        const unsigned long long add = b + o < kExtBins ? at[b + o] : 0ull;
        __syncthreads();
        if (b < kExtBins) at[b] += add;
        __syncthreads();
    }
    if (b < kExtBins && b > 0 && at[b] >= need && at[b + 1] < need) digit_s = (uint32_t)b;
    __syncthreads();
    const uint32_t d = digit_s;
    need -= at[d + 1];
    __syncthreads();
    return d;
}

// Counts of one level's digit contended on single words when every workgroup
// added to one histogram and the first level's few bins took every key one by
// one: 1e6 keys, 97 us of four passes with the host between them, now 22 with the list.
__global__ void __launch_bounds__(kExtSelBlock) k_key_hist(const uint32_t *keys, unsigned long long n, ExtSelect *sel,
                                                           int level)
{
    __shared__ uint32_t h[kExtBins];
    if (threadIdx.x < kExtBins) h[threadIdx.x] = 0u;
    unsigned long long need = sel->need[level - 1];
    const uint32_t prefix = (sel->prefix[level - 1] << 8) | select_digit(sel->hist[level - 1], need);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        sel->need[level] = need;
        sel->prefix[level] = prefix;
    }
    const int shift = 24 - 8 * level;
    for (unsigned long long i = (unsigned long long)blockIdx.x * kExtSelBlock + threadIdx.x; i < n;
         i += (unsigned long long)gridDim.x * kExtSelBlock) {
        const uint32_t k = keys[i];
        if ((k >> (shift + 8)) == prefix) atomicAdd(&h[(k >> shift) & 0xFFu], 1u);
    }
    flush_hist(h, sel->hist[level]);
}

// A workgroup's listed rows, passed on with one reservation (500 rows took one
// each, of one word, one after the other); those that do not fit reserve a place each.
struct ExtList {
    static constexpr unsigned N = 256;
    ExtRow rows[N];
    unsigned n;
    unsigned long long base;
    __device__ void add(const ExtRow &r, ExtRow *out, unsigned long long cap, unsigned long long *count)
    {
        const unsigned at = atomicAdd(&n, 1u);
        if (at < N) {
            rows[at] = r;
            return;
        }
        const unsigned long long pos = atomicAdd(count, 1ull);
        if (pos < cap) out[pos] = r;
    }
    __device__ void flush(ExtRow *out, unsigned long long cap, unsigned long long *count)
    {
        __syncthreads();
        const unsigned m = n < N ? n : N;
        if (threadIdx.x == 0 && m) base = atomicAdd(count, (unsigned long long)m);
        __syncthreads();
        for (unsigned i = threadIdx.x; i < m; i += kExtSelBlock)
            if (base + i < cap) out[base + i] = rows[i];
    }
};

__global__ void __launch_bounds__(kExtSelBlock) k_key_collect(const uint32_t *keys, const int *jmax,
                                                              unsigned long long n, ExtSelect *sel,
                                                              ExtRow *above, unsigned long long cap_above,
                                                              ExtRow *equal, unsigned long long cap_equal)
{
    __shared__ ExtList la, le;
    if (threadIdx.x == 0) la.n = le.n = 0u;
    unsigned long long need = sel->need[kExtLevels - 1];
    const uint32_t kth = (sel->prefix[kExtLevels - 1] << 8) | select_digit(sel->hist[kExtLevels - 1], need);
    if (blockIdx.x == 0 && threadIdx.x == 0) sel->out.need = need;
    for (unsigned long long i = (unsigned long long)blockIdx.x * kExtSelBlock + threadIdx.x; i < n;
         i += (unsigned long long)gridDim.x * kExtSelBlock) {
        const uint32_t k = keys[i];
        if (k < kth) continue;
        const ExtRow r{i, k, jmax[i]};
        if (k > kth)
            la.add(r, above, cap_above, &sel->out.above);
        else
            le.add(r, equal, cap_equal, &sel->out.equal);
    }
    la.flush(above, cap_above, &sel->out.above);
    le.flush(equal, cap_equal, &sel->out.equal);
}

__global__ void __launch_bounds__(kExtSelBlock) k_ext_begin(ExtSelect *sel, unsigned long long k)
{
    unsigned long long *w = reinterpret_cast<unsigned long long *>(sel);
    constexpr int n = sizeof(ExtSelect) / 8;
    const int i = blockIdx.x * kExtSelBlock + threadIdx.x;
    if (i < n) w[i] = w + i == &sel->need[0] ? k : 0ull;
}

}  // namespace

int ext_lds_bytes(int K) { return K >= 64 ? (K / 16) * 4 * (K / 32) * kWave * 16 : (K / 8) * (K / 4) * kWave * 16; }

template <int K>
hipError_t launch_grid_max_q(const ExtArgs &a, int n_cu, hipStream_t st)
{
    constexpr int lds = ExtQ<K>::TAB_BYTES, B = ExtQ<K>::BLOCK;
    auto kern = k_grid_max_q<K>;
    hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    int per_cu = 0;
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, B, lds);
    if (e != hipSuccess) return e;
    if (per_cu < 1) per_cu = 1;
    const unsigned long long chunks = (a.n + 15) / 16;
    unsigned long long grid = (unsigned long long)per_cu * n_cu;
    const unsigned long long want = (chunks + B / kWave - 1) / (B / kWave);
    if (want < grid) grid = want;
    if (grid < 1) grid = 1;
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(B), lds, st, a);
    return hipGetLastError();
}

hipError_t launch_grid_max(int K, const ExtArgs &a, int n_cu, hipStream_t st)
{
    if (K == 64) return launch_grid_max_q<64>(a, n_cu, st);
    if (K == 128) return launch_grid_max_q<128>(a, n_cu, st);
    const int lds = ext_lds_bytes(K);
    const unsigned long long tiles = (a.n + kTile - 1) / kTile;
    unsigned long long grid = (unsigned long long)n_cu * 4;
    const unsigned long long want = (tiles + kExtBlock / kWave - 1) / (kExtBlock / kWave);
    if (want < grid) grid = want;
    if (grid < 1) grid = 1;
#define TKDV_EXT(KK)                                                                                     \
    case KK: {                                                                                           \
        hipError_t e = hipFuncSetAttribute((const void *)k_grid_max<KK>,                                 \
                                           hipFuncAttributeMaxDynamicSharedMemorySize, lds);             \
        if (e != hipSuccess) return e;                                                                   \
        hipLaunchKernelGGL(k_grid_max<KK>, dim3((unsigned)grid), dim3(kExtBlock), lds, st, a);           \
        break;                                                                                           \
    }
    switch (K) {
        TKDV_EXT(8)
        TKDV_EXT(16)
        TKDV_EXT(32)
    default: return hipErrorInvalidValue;
    }
#undef TKDV_EXT
    return hipGetLastError();
}

hipError_t launch_ext_begin(ExtSelect *sel, unsigned long long k, hipStream_t st)
{
    constexpr unsigned g = (sizeof(ExtSelect) / 8 + kExtSelBlock - 1) / kExtSelBlock;
    hipLaunchKernelGGL(k_ext_begin, dim3(g), dim3(kExtSelBlock), 0, st, sel, k);
    return hipGetLastError();
}

hipError_t launch_ext_select(const uint32_t *keys, const int *jmax, unsigned long long n, ExtSelect *sel, ExtRow *above,
                             unsigned long long cap_above, ExtRow *equal, unsigned long long cap_equal, int n_cu,
                             hipStream_t st)
{
    unsigned long long g = (n + kExtSelBlock - 1) / kExtSelBlock;
    if (g > (unsigned long long)n_cu) g = n_cu;
    if (g < 1) g = 1;
    for (int level = 1; level < kExtLevels; ++level) {
        hipLaunchKernelGGL(k_key_hist, dim3((unsigned)g), dim3(kExtSelBlock), 0, st, keys, n, sel, level);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k_key_collect, dim3((unsigned)g), dim3(kExtSelBlock), 0, st, keys, jmax, n, sel, above, cap_above,
                       equal, cap_equal);
    return hipGetLastError();
}

}  // namespace tkdv
