// Full SRO evaluation on the matrix cores: descriptor and launcher.
#pragma once

#include <hip/hip_runtime.h>

#include "geometry.h"

namespace pyhea {

constexpr int kMfmaTiles = 14;     // (column, layer) displacements of a launch at most
constexpr int kMfmaGroups = kMaxShells + 1;   // sums per configuration: the shells, and each site with itself
// cells a workgroup may count: a displacement's sums of 16 * 4 quarter units per cell stay below 2^24
// (and kQuarter + sum at most 2^22)
constexpr int kMfmaMaxCells = 1 << 16;

// Feature sums are whole numbers of quarters: a pair that counts 1 weighs up to 64.  A
// workgroup's (at most 4 sublattices x 12 neighbours x kMfmaMaxCells pairs, 2^27.6) fit 32
// bits.  A configuration's, up to 32 N z, do not where N z >= 2^26, and since they are
// divided on the way to counts they must not wrap: 64 bits.
typedef int32_t MfmaGroupSum;
typedef int64_t MfmaSum;

// a_i of species i < 4 from four feature sums doubled (f' = 2 f)
template <class Sum>
__host__ __device__ inline void species_of_features(Sum f0, Sum f1, Sum f2, Sum f3, Sum *a) {
    a[3] = (f3 - f1 - f2) / 2;
    a[0] = f0;
    a[1] = f1 / 2 - a[3];
    a[2] = f2 / 4 - a[3];
}

struct MfmaDesc {
    int32_t Lx, Ly, Lz, M, S;
    int32_t W;          // words per column: word q, nibble p holds layer W p + q - dead
    int32_t NP;         // nibbles of a word in use
    int32_t dead;       // slots below layer 0, W NP - Lz
    int32_t xs;         // columns per quarter of a row
    int32_t Xs, RS;     // fragments between sublattices / rows in LDS
    int32_t ys;         // centre rows per workgroup
    int32_t R;          // rows a workgroup holds (its centre rows and one above, or all)
    int32_t nchunks;    // workgroups per configuration
    int32_t threads, lds_bytes;
    int32_t tiles;      // 14 or 10 (FCC), 6 (BCC)
    int32_t even;       // quarters of a row and groups of 4 rows are whole
    int32_t step;       // configurations per launch
    int32_t whole;      // the wavefronts' shares are whole rows
    uint32_t N;
    double inv_xs, inv_R;   // 1 / xs, 1 / R
    uint32_t codes_lo, codes_hi;   // code of species 0-3 and 4-7 (8: invalid)
    int32_t zk[kMaxShells];
    uint8_t list[kMfmaTiles * 16];       // 16 * tile + 4 * row class + column class, by group
    uint8_t start[kMfmaGroups + 1];
};

// Fills md; false if the matrix-core kernel does not cover the geometry (it covers 2 to 5
// species, FCC shells 1-4 and BCC shells 1-3) or is not the faster one there.
bool fill_mfma_desc(const Geometry &g, int lds_budget, int64_t K, MfmaDesc *md);
// Configurations one launch takes: a grid holds less than 2^32 threads, and a
// configuration's workgroups lie eight blocks apart.
constexpr int64_t mfma_configs_per_launch(int threads, int nchunks) {
    return ((int64_t(1) << 32) - 1) / threads / nchunks / 8 * 8;
}

// int32 of scratch per workgroup of a configuration that spans several
constexpr int kMfmaPartial = kMfmaGroups * 16 + 4;

size_t mfma_partial_bytes(const MfmaDesc &md, int64_t K);

// As launch_count_bits; `partial` holds mfma_partial_bytes.
hipError_t launch_count_mfma(const MfmaDesc &md, int64_t K, const int8_t *species, int32_t *partial, int32_t *counts,
                             int32_t *bad, const double *tw, double *S_F, hipStream_t stream);

}  // namespace pyhea
