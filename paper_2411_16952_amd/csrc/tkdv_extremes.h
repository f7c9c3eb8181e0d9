// Extreme wave fields among stored samples: launchers shared with the C ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace tkdv {

constexpr int kExtBlock = 256;  // threads per workgroup of k_grid_max (K <= 32)

constexpr int kExtSelBlock = 1024;  // threads per workgroup of the selection's kernels
constexpr int kExtBins = 256, kExtLevels = 4;  // the selection's digits of 8 bits, from the top
constexpr int kExtShards = 8;   // copies of a level's counts, one for a workgroup in eight

// The selection of the k-th largest key, on the device from start to end.
struct ExtSelect {
    unsigned long long hist[kExtLevels][kExtShards * kExtBins];  // by digit, of the keys that share the prefix
    unsigned long long need[kExtLevels];  // rows still to take at or below the prefix of `level` digits
    uint32_t prefix[kExtLevels];
    struct Out {
        unsigned long long n_exceed;      // rows above the threshold
        unsigned long long above, equal;  // rows above the k-th key, rows equal to it
        unsigned long long need;          // of the equal ones, how many to take
    } out;
};
// A listed row.
struct ExtRow {
    unsigned long long row;
    uint32_t key;
    int j;
};

struct ExtArgs {
    const float *xhat;          // [n][stride] rows of x^ (first 2K entries used)
    unsigned long long n, stride;
    const void *phi_f32;        // FP32 synthesis tables of K (K = 64, 128: quarter-period statistics tables)
    float amp;                  // sqrt(2 E0/pi)
    float threshold;            // rows with max u above it are counted
    uint32_t *keys;             // [n] order-preserving keys of the maxima
    float *umax;                // [n] or nullptr
    int *jmax;                  // [n] or nullptr
    unsigned long long *n_exceed;
    unsigned long long *hist;   // the first level's counts (ExtSelect)
};

int ext_lds_bytes(int K);
hipError_t launch_grid_max(int K, const ExtArgs &a, int n_cu, hipStream_t st);
hipError_t launch_ext_begin(ExtSelect *sel, unsigned long long k, hipStream_t st);
// The rows above the k-th largest key (at most cap_above listed, in any order)
// and equal to it (cap_equal), after launch_grid_max.
hipError_t launch_ext_select(const uint32_t *keys, const int *jmax, unsigned long long n, ExtSelect *sel, ExtRow *above,
                             unsigned long long cap_above, ExtRow *equal, unsigned long long cap_equal, int n_cu,
                             hipStream_t st);

}  // namespace tkdv
