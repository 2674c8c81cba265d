// Launchers of the pyhea kernels.
#pragma once

#include <hip/hip_runtime.h>

#include "geometry.h"

namespace pyhea {

constexpr int kMaxLookahead = 8;   // pyhea_tune_force_lookahead: 1 = step by step, more = quiet steps in windows
constexpr int kRing = 8;           // steps whose candidates are drawn ahead
constexpr int kChunk = 32;         // members of a commit chunk at most (half a wavefront)
constexpr int kMaxWaves = 8;       // wavefronts of a chain's workgroup at most

// LDS of the MC kernel without the species store: CH = members of a commit chunk.
int mc_lds_bytes(int S, int M, int B, int CH);

// bytes of the species store for a padded chain
inline int64_t species_store_bytes(int store, int64_t Npad) {
    if (store == kStoreLds8) return (Npad + 15) & ~int64_t(15);
    if (store == kStoreLds4) return (((Npad + 7) / 8) * 4 + 15) & ~int64_t(15);
    return 0;
}

// Raises a kernel's dynamic LDS limit to at least `lds` bytes on the current
// device; remembers what it set, so repeated launches make no runtime call.
hipError_t set_max_lds(const void *fn, size_t lds);

// One launch of n_chains chains (one block each) for up to max_steps steps.
// quiet > 0 (chains with image or pad_global, scan_nulls and scan_cap set): a
// chain also ends its launch, with a window to scan, once `quiet` steps in a row
// committed nothing.
hipError_t launch_mc(const ChainDesc *descs_dev, int n_chains, int store, int M, int B, int waves, int K, int CH,
                     int lds_bytes, int max_steps, hipStream_t stream, int quiet = 0);

// The windows of quiet chains (chains without one are skipped), each by
// blocks_per_chain blocks; store_bytes: the largest LDS store of the chains.
constexpr int kScanThreads = 512;
int scan_lds_bytes(int S, int M);
hipError_t launch_scan(const ChainDesc *descs_dev, int n_chains, int store, int M, int store_bytes, int S,
                       int blocks_per_chain, hipStream_t stream);
// Ratio tables of chains from their initial counts (descriptor order; bad [n]
// the invalid-id flags in the same order); invalid chains get status EINVAL.
hipError_t launch_chain_ratio(const ChainDesc *descs_dev, int n_chains, const int32_t *bad, hipStream_t stream);
hipError_t launch_pad_fill(const ChainDesc *descs_dev, int n_chains, hipStream_t stream);
hipError_t launch_pad_drain(const ChainDesc *descs_dev, int n_chains, hipStream_t stream);
// out[i] = *descs_dev[i].state (device array of n_chains states).
hipError_t launch_gather_states(const ChainDesc *descs_dev, int n_chains, ChainState *out, hipStream_t stream);
// S and F of every chain's maintained counts into its state (Eq. 2-3).
hipError_t launch_final_objective(const ChainDesc *descs_dev, int n_chains, hipStream_t stream);

// Full evaluation: pair counts of K configurations of one geometry.
struct EvalDesc {
    int32_t A, lgA, Lx, Ly, Lz, M, S;
    int32_t n_half;                       // offsets with one of each +-d pair
    int32_t z0;                           // coordination number of shell 1
    int32_t zk[kMaxShells];
    double inv_Lx, inv_Ly;
    uint32_t N;
    int32_t Z;                            // all offsets of shells 1..S
    // per (basis, half offset): dcx, dcy, dcz, target basis, shell (int8 each)
    int8_t half[4][kMaxOffsets / 2][5];
    int8_t off[kMaxOffsets][4];           // dx, dy, dz, shell (half units)
};

void fill_eval_desc(const Geometry &g, EvalDesc *d);

// One configuration of a many-chain count launch (each its own geometry).
struct CountTask {
    EvalDesc ed;
    const int8_t *species;  // N sites, unpadded
    int32_t *counts;        // [S][M][M], zero before the launch
    int32_t *bad;           // set to 1 if a species id lies outside [0, M); zero before the launch
};
// Sites per workgroup of the many-configuration count: 2048, halved (down to
// 256) while the launch would have fewer than 2048 workgroups, so that a few
// small configurations still spread over the chip.
inline uint32_t count_tile_for(uint64_t total_sites) {
    uint32_t tile = 2048;
    while (tile > 256 && total_sites < (uint64_t)tile * 2048) tile >>= 1;
    return tile;
}
inline uint32_t count_tiles(uint32_t N, uint32_t tile) { return (N + tile - 1) / tile; }

// Pair counts of n configurations with different geometries in one launch.
// tile0[c] = first tile of task c (prefix sums of count_tiles(N, tile)),
// n_tiles = total; max_E = the largest S M M of the tasks (LDS histograms).
hipError_t launch_count_tasks(const CountTask *tasks, const uint32_t *tile0, int n, uint32_t n_tiles, uint32_t tile,
                              int max_E, hipStream_t stream);

hipError_t launch_zero_i32(int32_t *p, int64_t n, hipStream_t stream);

// Target and weight tables (at most S M M + S doubles) copied to the device by a
// kernel whose arguments carry them: stream-ordered, and the host never waits.
constexpr int kMaxTable = kMaxShells * kMaxSpecies * kMaxSpecies + kMaxShells;
struct SmallTable {
    double v[kMaxTable];
};
hipError_t launch_upload(const SmallTable &t, int n, double *dst, hipStream_t stream);

hipError_t launch_count_gather(const EvalDesc &ed, int64_t K, const int8_t *species,
                               int32_t *counts, int32_t *bad, hipStream_t stream);
// S_F [K][2] from counts.
hipError_t launch_objective_epilogue(const EvalDesc &ed, int64_t K, const int32_t *counts,
                                     const int32_t *bad, const double *target, const double *weight,
                                     double *S_F, hipStream_t stream);
// Eq. 2-3 of one configuration into page-locked host memory; a zero table gives the alpha
// alone (S and F then mean nothing).
struct OneDesc {
    uint32_t N;
    int32_t M, S;
    int32_t zk[kMaxShells];
};
struct OneResult {
    double S_F[2];
    double alpha[kMaxShells * kMaxSpecies * kMaxSpecies];
    int32_t counts[kMaxShells * kMaxSpecies * kMaxSpecies];
    int32_t invalid;   // an id out of range or a species absent: only this is set
};
hipError_t launch_objective_one(const OneDesc &od, const SmallTable &tw, const int32_t *counts, const int32_t *bad,
                                OneResult *out, hipStream_t stream);
// Row r of dst [count][N] becomes row rows[r] of src (N < 2^32; no overlap).
constexpr int kCopyRows = 256;
struct RowTable {
    int32_t row[kCopyRows];
};
hipError_t launch_copy_rows(const int *rows, int count, int64_t N, const int8_t *src, int8_t *dst, hipStream_t stream);
// `status` is host memory: 1 if an id is invalid or a species absent (nothing else is
// written then), else 0.
hipError_t launch_trial_eval(const EvalDesc &ed, const SmallTable &tw, const int8_t *species, const int32_t *counts,
                             const int32_t *bad, int64_t n_pairs, const int32_t *pairs, double *dS, int32_t *dN,
                             int32_t *status, hipStream_t stream);
// Non-incremental baseline: out[i] = base with sites pairs[i] swapped (out
// [n][N]); *bad |= 1 for a pair outside [0, N).  dS[i] = S_F[i][0] - S0[0].
hipError_t launch_swap_copies(const int8_t *base, int64_t N, const int32_t *pairs, int n, int8_t *out, int32_t *bad,
                              hipStream_t stream);
hipError_t launch_sub_objective(const double *S_F, const double *S0, int n, double *dS, hipStream_t stream);

// Random solutions of the global search: configuration c of n_configs is pool
// slot d.slot0 + c (out [n_configs][N]); d.prefix[j] = sum of the first j
// species counts (prefix[M] = N).
struct RandomConfigDesc {
    uint64_t seed;
    uint32_t iteration;
    uint32_t slot0;
    int32_t M;
    uint32_t prefix[9];
};
hipError_t launch_random_configs(uint32_t N, const RandomConfigDesc &d, int n_configs, int8_t *out,
                                 hipStream_t stream);

hipError_t launch_philox(const uint32_t *ctr, uint64_t seed, int64_t n, uint32_t *out,
                         hipStream_t stream);

}  // namespace pyhea
