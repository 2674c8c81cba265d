// Full SRO evaluation kernels (Sec. 4.3, Eq. 2; Sec. 4.4, Eq. 3), the
// per-swap evaluation API (Sec. 4.5, Eq. 4) and a device Philox stream.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>

#include "device_common.h"
#include "mc_kernels.h"

namespace pyhea {

void fill_eval_desc(const Geometry &g, EvalDesc *d) {
    std::memset(d, 0, sizeof(*d));
    d->A = g.A;
    d->lgA = g.lgA;
    d->Lx = g.L[0];
    d->Ly = g.L[1];
    d->Lz = g.L[2];
    d->M = g.M;
    d->S = g.S;
    d->z0 = g.z[0];
    for (int k = 0; k < kMaxShells; ++k) d->zk[k] = k < g.S ? g.z[k] : 0;
    d->inv_Lx = 1.0 / (double)g.L[0];
    d->inv_Ly = 1.0 / (double)g.L[1];
    d->N = (uint32_t)g.N;
    d->Z = g.Z;
    int nh = 0;
    for (int t = 0; t < g.Z; ++t) {
        int shell = 0;
        while (t >= g.zstart[shell + 1]) ++shell;
        const int dx = g.off[t][0], dy = g.off[t][1], dz = g.off[t][2];
        d->off[t][0] = (int8_t)dx;
        d->off[t][1] = (int8_t)dy;
        d->off[t][2] = (int8_t)dz;
        d->off[t][3] = (int8_t)shell;
        // keep one offset of each +-d pair
        const bool keep = dz > 0 || (dz == 0 && (dy > 0 || (dy == 0 && dx > 0)));
        if (!keep) continue;
        for (int b = 0; b < g.A; ++b) {
            int dc[3], bt;
            offset_target(g, b, t, dc, &bt);
            d->half[b][nh][0] = (int8_t)dc[0];
            d->half[b][nh][1] = (int8_t)dc[1];
            d->half[b][nh][2] = (int8_t)dc[2];
            d->half[b][nh][3] = (int8_t)bt;
            d->half[b][nh][4] = (int8_t)shell;
        }
        ++nh;
    }
    d->n_half = nh;
}

namespace {

__device__ __forceinline__ int wrap1(int v, int L) {
    while (v < 0) v += L;
    while (v >= L) v -= L;
    return v;
}

// Pair counts by gather: every site visits one offset of each +-d pair,
// N[k][i][j] = H[k][i][j] + H[k][j][i] with H the half counts (the map
// p -> p - d is a bijection of the periodic cell).  LDS-privatised int32
// histogram per workgroup, merged into global counts with one atomic per bin.
__global__ void __launch_bounds__(256) count_gather_kernel(EvalDesc ed, int64_t K,
                                                           const int8_t *__restrict__ species,
                                                           int32_t *__restrict__ counts,
                                                           int32_t *__restrict__ bad) {
    __shared__ int32_t hist[kMaxShells * kMaxSpecies * kMaxSpecies];
    __shared__ int32_t bad_sh;
    const int M = ed.M, E = ed.S * ed.M * ed.M;
    for (int64_t kc = blockIdx.y; kc < K; kc += gridDim.y) {
        for (int e = threadIdx.x; e < E; e += blockDim.x) hist[e] = 0;
        if (threadIdx.x == 0) bad_sh = 0;
        __syncthreads();
        const int8_t *sp = species + kc * (int64_t)ed.N;
        for (uint32_t p = blockIdx.x * blockDim.x + threadIdx.x; p < ed.N; p += gridDim.x * blockDim.x) {
            const int s = sp[p];
            if (s < 0 || s >= M) {
                bad_sh = 1;
                continue;
            }
            const SiteCoord c = site_coord(p, ed.lgA, ed.Lx, ed.Ly, ed.inv_Lx, ed.inv_Ly);
            for (int hh = 0; hh < ed.n_half; ++hh) {
                const int8_t *o = ed.half[c.b][hh];
                const int x = wrap1(c.cx + o[0], ed.Lx);
                const int y = wrap1(c.cy + o[1], ed.Ly);
                const int z = wrap1(c.cz + o[2], ed.Lz);
                const int s2 = sp[((z * ed.Ly + y) * ed.Lx + x) * ed.A + o[3]];
                if (s2 < 0 || s2 >= M) continue;
                atomicAdd(&hist[(o[4] * M + s) * M + s2], 1);
            }
        }
        __syncthreads();
        for (int e = threadIdx.x; e < E; e += blockDim.x) {
            const int kk = e / (M * M), i = (e / M) % M, j = e % M;
            const int v = hist[e] + hist[(kk * M + j) * M + i];
            if (v) atomicAdd(&counts[kc * E + e], v);
        }
        if (threadIdx.x == 0 && bad_sh) atomicOr(&bad[kc], 1);
        __syncthreads();
    }
}

// The same gather count for many configurations of different geometries: the
// grid is the concatenation of every configuration's site tiles.  The LDS
// histogram has kHistCopies interleaved copies (bin e, copy c at e * kHistCopies
// + c; lane l adds into copy l mod kHistCopies), so lanes of a wavefront that
// hit the same bin hit different words.
constexpr int kHistCopies = 16;
__global__ void __launch_bounds__(256) count_tasks_kernel(const CountTask *__restrict__ tasks,
                                                          const uint32_t *__restrict__ tile0, int n, uint32_t tile) {
    extern __shared__ int32_t hist[];   // [E][kHistCopies], then the invalid-id flag
    // owning configuration: the last c with tile0[c] <= blockIdx.x
    int lo = 0, hi = n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (tile0[mid] <= blockIdx.x)
            lo = mid;
        else
            hi = mid - 1;
    }
    const CountTask &t = tasks[lo];
    const EvalDesc &ed = t.ed;
    const int M = ed.M, E = ed.S * ed.M * ed.M;
    int32_t *bad_sh = hist + E * kHistCopies;
    for (int e = threadIdx.x; e <= E * kHistCopies; e += blockDim.x) hist[e] = 0;
    __syncthreads();
    const int8_t *sp = t.species;
    const int copy = threadIdx.x % kHistCopies;
    const uint32_t p0 = (blockIdx.x - tile0[lo]) * tile;
    const uint32_t p1 = min(p0 + tile, ed.N);
    for (uint32_t p = p0 + threadIdx.x; p < p1; p += blockDim.x) {
        const int s = sp[p];
        if (s < 0 || s >= M) {
            *bad_sh = 1;
            continue;
        }
        const SiteCoord c = site_coord(p, ed.lgA, ed.Lx, ed.Ly, ed.inv_Lx, ed.inv_Ly);
        for (int hh = 0; hh < ed.n_half; ++hh) {
            const int8_t *o = ed.half[c.b][hh];
            const int x = wrap1(c.cx + o[0], ed.Lx);
            const int y = wrap1(c.cy + o[1], ed.Ly);
            const int z = wrap1(c.cz + o[2], ed.Lz);
            const int s2 = sp[((z * ed.Ly + y) * ed.Lx + x) * ed.A + o[3]];
            if (s2 < 0 || s2 >= M) continue;
            atomicAdd(&hist[((o[4] * M + s) * M + s2) * kHistCopies + copy], 1);
        }
    }
    __syncthreads();
    for (int e = threadIdx.x; e < E; e += blockDim.x) {
        const int kk = e / (M * M), i = (e / M) % M, j = e % M;
        const int eT = (kk * M + j) * M + i;
        int v = 0;
        for (int q = 0; q < kHistCopies; ++q) v += hist[e * kHistCopies + q] + hist[eT * kHistCopies + q];
        if (v) atomicAdd(&t.counts[e], v);
    }
    if (threadIdx.x == 0 && *bad_sh) atomicOr(t.bad, 1);
}

__global__ void upload_kernel(SmallTable t, int n, double *__restrict__ dst) {
    for (int i = threadIdx.x; i < n; i += blockDim.x) dst[i] = t.v[i];
}

__global__ void zero_i32_kernel(int32_t *p, int64_t n) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0;
}

// alpha / S / F of Eq. 2-3 per configuration (one thread per configuration),
// binary64, no contraction: R = N / (n_i n_j z_k), alpha = 1 - N_ij R,
// Q_k = sum_i (sum_j (alpha - t)^2), S = sum_k w_k Q_k, F = sqrt(S).
__global__ void objective_kernel(EvalDesc ed, int64_t K, const int32_t *__restrict__ counts,
                                 const int32_t *__restrict__ bad, const double *__restrict__ target,
                                 const double *__restrict__ weight, double *__restrict__ S_F) {
    const int64_t kc = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (kc >= K) return;
    const int M = ed.M, E = ed.S * M * M;
    const int32_t *c = counts + kc * E;
    int64_t n[kMaxSpecies];
    bool ok = bad[kc] == 0;
    for (int i = 0; i < M; ++i) {
        int64_t r = 0;
        for (int j = 0; j < M; ++j) r += c[i * M + j];
        n[i] = r / ed.z0;
        ok = ok && n[i] > 0;
    }
    if (!ok) {
        S_F[2 * kc] = __longlong_as_double(0x7ff8000000000000ll);
        S_F[2 * kc + 1] = __longlong_as_double(0x7ff8000000000000ll);
        return;
    }
    double sum = 0.0;
    for (int k = 0; k < ed.S; ++k) {
        double Q = 0.0;
        for (int i = 0; i < M; ++i) {
            double row = 0.0;
            for (int j = 0; j < M; ++j) {
                const int e = (k * M + i) * M + j;
                const double R = (double)ed.N / (double)(n[i] * n[j] * (int64_t)ed.zk[k]);
                const double a = 1.0 - (double)c[e] * R;
                const double dd = a - target[e];
                row = row + dd * dd;
            }
            Q = Q + row;
        }
        sum = sum + weight[k] * Q;
    }
    S_F[2 * kc] = sum;
    S_F[2 * kc + 1] = sqrt(sum);
}

// objective_kernel for a few configurations: one 64-thread block per
// configuration, its entries spread over the lanes and its rows summed by one
// lane each, then the rows into Q_k and S by lane 0 -- the same expressions and
// summation order as objective_kernel, so the results are the same bit for bit.
__global__ void __launch_bounds__(64) objective_block_kernel(EvalDesc ed, const int32_t *__restrict__ counts,
                                                             const int32_t *__restrict__ bad,
                                                             const double *__restrict__ target,
                                                             const double *__restrict__ weight,
                                                             double *__restrict__ S_F) {
    __shared__ int64_t n[kMaxSpecies];
    __shared__ double lsq[kMaxShells * kMaxSpecies * kMaxSpecies];
    __shared__ double lrow[kMaxShells * kMaxSpecies];
    const int64_t kc = blockIdx.x;
    const int tid = (int)threadIdx.x;
    const int M = ed.M, E = ed.S * M * M;
    const int32_t *c = counts + kc * E;
    if (tid < M) {
        int64_t r = 0;
        for (int j = 0; j < M; ++j) r += c[tid * M + j];
        n[tid] = r / ed.z0;
    }
    __syncthreads();
    bool ok = bad[kc] == 0;
    for (int i = 0; i < M; ++i) ok = ok && n[i] > 0;
    if (!ok) {
        if (tid == 0) {
            S_F[2 * kc] = __longlong_as_double(0x7ff8000000000000ll);
            S_F[2 * kc + 1] = __longlong_as_double(0x7ff8000000000000ll);
        }
        return;
    }
    for (int e = tid; e < E; e += blockDim.x) {
        const int k = e / (M * M), i = (e / M) % M, j = e % M;
        const double R = (double)ed.N / (double)(n[i] * n[j] * (int64_t)ed.zk[k]);
        const double a = 1.0 - (double)c[e] * R;
        const double dd = a - target[e];
        lsq[e] = dd * dd;
    }
    __syncthreads();
    for (int r = tid; r < ed.S * M; r += blockDim.x) {
        double row = 0.0;
        for (int j = 0; j < M; ++j) row = row + lsq[r * M + j];
        lrow[r] = row;
    }
    __syncthreads();
    if (tid == 0) {
        double sum = 0.0;
        for (int k = 0; k < ed.S; ++k) {
            double Q = 0.0;
            for (int i = 0; i < M; ++i) Q = Q + lrow[k * M + i];
            sum = sum + weight[k] * Q;
        }
        S_F[2 * kc] = sum;
        S_F[2 * kc + 1] = sqrt(sum);
    }
}

// Eq. 2-3 of a single configuration whose results the host waits for: the target and
// weights arrive with the arguments and the results go to page-locked host memory, so that
// nothing is uploaded or read back (a launch, a copy and its staging: 30 us of a call).
// Expressions and summation order of objective_block_kernel.
constexpr int kOneThreads = 256;   // S M^2 entries at once
__global__ void __launch_bounds__(kOneThreads)
objective_one_kernel(OneDesc od, SmallTable tw, const int32_t *__restrict__ counts, const int32_t *__restrict__ bad,
                     OneResult *__restrict__ out) {
    __shared__ int32_t c[kMaxShells * kMaxSpecies * kMaxSpecies];
    __shared__ int64_t n[kMaxSpecies];
    __shared__ double lsq[kMaxShells * kMaxSpecies * kMaxSpecies];
    __shared__ double lrow[kMaxShells * kMaxSpecies];
    const int tid = (int)threadIdx.x;
    const int M = od.M, E = od.S * M * M;
    const int isbad = *bad;
    if (tid < E) {
        c[tid] = counts[tid];
        out->counts[tid] = c[tid];
    }
    __syncthreads();
    if (tid < M) {
        int64_t r = 0;
        for (int j = 0; j < M; ++j) r += c[tid * M + j];
        n[tid] = r / od.zk[0];
    }
    __syncthreads();
    bool ok = isbad == 0;
    for (int i = 0; i < M; ++i) ok = ok && n[i] > 0;
    if (tid == 0) out->invalid = ok ? 0 : 1;
    if (!ok) return;
    if (tid < E) {
        const int k = tid / (M * M), i = (tid / M) % M, j = tid % M;
        const double R = (double)od.N / (double)(n[i] * n[j] * (int64_t)od.zk[k]);
        const double a = 1.0 - (double)c[tid] * R;
        out->alpha[tid] = a;
        const double dd = a - tw.v[tid];
        lsq[tid] = dd * dd;
    }
    __syncthreads();
    if (tid < od.S * M) {
        double row = 0.0;
        for (int j = 0; j < M; ++j) row = row + lsq[tid * M + j];
        lrow[tid] = row;
    }
    __syncthreads();
    if (tid == 0) {
        double sum = 0.0;
        for (int k = 0; k < od.S; ++k) {
            double Q = 0.0;
            for (int i = 0; i < M; ++i) Q = Q + lrow[k * M + i];
            sum = sum + tw.v[E + k] * Q;
        }
        out->S_F[0] = sum;
        out->S_F[1] = sqrt(sum);
    }
}

// Eq. 2-3 on a chain's maintained counts, binary64 in the host contract's order
// (alpha = 1 - N R, (alpha - t)^2 summed along a row, rows into Q_k, S = sum_k
// w_k Q_k), written to its state with F = sqrt(S).  One thread per chain.
__global__ void final_objective_kernel(const ChainDesc *__restrict__ descs, int n) {
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= n) return;
    const ChainDesc &d = descs[c];
    const int M = d.M;
    double sum = 0.0;
    for (int k = 0; k < d.S; ++k) {
        double Q = 0.0;
        for (int i = 0; i < M; ++i) {
            double row = 0.0;
            for (int j = 0; j < M; ++j) {
                const int e = (k * M + i) * M + j;
                const double a = 1.0 - (double)d.counts[e] * d.R[e];
                const double dd = a - d.target[e];
                row = row + dd * dd;
            }
            Q = Q + row;
        }
        sum = sum + d.w[k] * Q;
    }
    d.state->S = sum;
    d.state->F = sqrt(sum);
}

// site id of position (x, y, z) in half units, wrapped into the box
__device__ __forceinline__ int32_t site_at(const EvalDesc &ed, int x, int y, int z) {
    x = wrap1(x, 2 * ed.Lx);
    y = wrap1(y, 2 * ed.Ly);
    z = wrap1(z, 2 * ed.Lz);
    int b;
    const int px = x & 1, py = y & 1, pz = z & 1;
    if (ed.A == 4)
        b = (px && py) ? 1 : (px && pz) ? 2 : (py && pz) ? 3 : 0;
    else
        b = px;
    return (((z >> 1) * ed.Ly + (y >> 1)) * ed.Lx + (x >> 1)) * ed.A + b;
}

// What no swap changes, made once per workgroup: R, the targets, the old terms.
struct TrialTables {
    int64_t n[kMaxSpecies];
    int32_t off[kMaxOffsets], cnt[kMaxShells * kMaxSpecies * kMaxSpecies];
    double R[kMaxShells * kMaxSpecies * kMaxSpecies], t[kMaxShells * kMaxSpecies * kMaxSpecies];
    double old_sq[kMaxShells * kMaxSpecies * kMaxSpecies], weight[kMaxShells];
};

// Fills l; false if an id is invalid or a species absent (*status, in host memory, is then 1
// and nothing else is to be written; else 0).
__device__ __forceinline__ bool trial_tables(TrialTables &l, const EvalDesc &ed, const SmallTable &tw,
                                             const int32_t *counts, const int32_t *bad, int32_t *status) {
    const int M = ed.M, E = ed.S * M * M;
    const int tid = (int)threadIdx.x, nthreads = (int)blockDim.x;
    if (tid < M) {
        int64_t r = 0;
        for (int j = 0; j < M; ++j) r += counts[tid * M + j];
        l.n[tid] = r / ed.z0;
    }
    for (int i = tid; i < ed.Z; i += nthreads) __builtin_memcpy(&l.off[i], ed.off[i], 4);
    if (tid < ed.S) l.weight[tid] = tw.v[E + tid];
    __syncthreads();
    bool ok = *bad == 0;
    for (int i = 0; i < M; ++i) ok = ok && l.n[i] > 0;
    if (blockIdx.x == 0 && tid == 0) *status = ok ? 0 : 1;
    if (!ok) return false;
    for (int e = tid; e < E; e += nthreads) {
        const int k = e / (M * M), i = (e / M) % M, j = e % M;
        l.cnt[e] = counts[e];
        l.t[e] = tw.v[e];
        l.R[e] = (double)ed.N / (double)(l.n[i] * l.n[j] * (int64_t)ed.zk[k]);
        const double a0 = 1.0 - (double)counts[e] * l.R[e];
        const double d0 = a0 - tw.v[e];
        l.old_sq[e] = d0 * d0;
    }
    __syncthreads();
    return true;
}

// dN_ij of a shell for swapping species a != b, from the changes D of the neighbours'
// species (of the site that becomes a, less those of the site that becomes b).
__device__ __forceinline__ int trial_dn(int i, int j, int a, int b, int Da, int Db, int Di, int Dj) {
    if (i == a) return j == a ? 2 * Da : (j == b ? Db - Da : Dj);
    if (i == b) return j == b ? -2 * Db : (j == a ? Db - Da : -Dj);
    return j == a ? Di : (j == b ? -Di : 0);
}

// dS and dN of given swaps against one configuration (no swap applied).  Half a
// wavefront takes a pair: its lanes read the neighbours of both sites at once and add up
// the change of the rows of species a and b in LDS; then a lane per row of a shell sums its
// M terms and one lane the rows, in the order of Eq. 3.  A lane per pair took 83 us for
// 4,096 pairs on FCC 20^3, 5 species, 3 shells: 42 dependent reads twice, row counters in
// scratch memory and 75 divisions per pair; now the call, count included, takes 59 us of
// 273.  Bound by the latency of those steps and the launches.
constexpr int kTrialLanes = 32;      // a lane for each of S M rows
constexpr int kTrialThreads = 256;
__global__ void __launch_bounds__(kTrialThreads)
trial_eval_kernel(EvalDesc ed, SmallTable tw, const int8_t *__restrict__ sp, const int32_t *__restrict__ counts,
                  const int32_t *__restrict__ bad, int64_t n_pairs, const int32_t *__restrict__ pairs,
                  double *__restrict__ dS_out, int32_t *__restrict__ dN_out, int32_t *__restrict__ status) {
    constexpr int kGroups = kTrialThreads / kTrialLanes;
    __shared__ TrialTables l;
    __shared__ int32_t D_all[kGroups][kMaxShells][kMaxSpecies];
    __shared__ double row_all[kGroups][kMaxShells * kMaxSpecies];
    const int M = ed.M, E = ed.S * M * M;
    const int tid = (int)threadIdx.x;
    if (!trial_tables(l, ed, tw, counts, bad, status)) return;
    const int group = tid / kTrialLanes, lane = tid % kTrialLanes;
    int32_t(&D)[kMaxShells][kMaxSpecies] = D_all[group];
    double *row = row_all[group];
    // every group of a workgroup makes the same number of turns, for the barriers
    for (int64_t u0 = (int64_t)blockIdx.x * kGroups; u0 < n_pairs; u0 += (int64_t)gridDim.x * kGroups) {
        const int64_t u = u0 + group;
        const bool here = u < n_pairs;
        const int32_t p = here ? pairs[2 * u] : -1, q = here ? pairs[2 * u + 1] : -1;
        const bool valid = here && p >= 0 && q >= 0 && (uint32_t)p < ed.N && (uint32_t)q < ed.N;
        (&D[0][0])[lane] = 0;
        __syncthreads();
        int a = 0, b = 0;
        if (valid) {
            a = sp[p];
            b = sp[q];
            if (a != b) {
                const SiteCoord c = site_coord((uint32_t)p, ed.lgA, ed.Lx, ed.Ly, ed.inv_Lx, ed.inv_Ly);
                const SiteCoord d = site_coord((uint32_t)q, ed.lgA, ed.Lx, ed.Ly, ed.inv_Lx, ed.inv_Ly);
                int bx, by, bz, ex, ey, ez;
                basis_bits(ed.A, c.b, bx, by, bz);
                basis_bits(ed.A, d.b, ex, ey, ez);
                for (int i = lane; i < ed.Z; i += kTrialLanes) {
                    const int32_t o = l.off[i];
                    const int ox = (int8_t)o, oy = (int8_t)(o >> 8), oz = (int8_t)(o >> 16), k = o >> 24;
                    const int32_t rp = site_at(ed, 2 * c.cx + bx + ox, 2 * c.cy + by + oy, 2 * c.cz + bz + oz);
                    const int32_t rq = site_at(ed, 2 * d.cx + ex + ox, 2 * d.cy + ey + oy, 2 * d.cz + ez + oz);
                    if (rp != q) atomicAdd(&D[k][sp[rp]], -1);
                    if (rq != p) atomicAdd(&D[k][sp[rq]], 1);
                }
            }
        }
        __syncthreads();
        if (valid && lane < ed.S * M) {
            const int k = lane / M, i = lane - k * M;
            const int Da = D[k][a], Db = D[k][b], Di = D[k][i];
            double rowsum = 0.0;
            for (int j = 0; j < M; ++j) {
                const int dn = a != b ? trial_dn(i, j, a, b, Da, Db, Di, D[k][j]) : 0;
                const int e = lane * M + j;
                if (dN_out) dN_out[u * E + e] = dn;
                const double a1 = 1.0 - (double)(l.cnt[e] + dn) * l.R[e];
                const double d1 = a1 - l.t[e];
                rowsum = rowsum + (d1 * d1 - l.old_sq[e]);
            }
            row[lane] = rowsum;
        }
        __syncthreads();
        if (here && lane == 0) {
            double acc = 0.0;
            for (int k = 0; k < ed.S; ++k) {
                double dQ = 0.0;
                for (int i = 0; i < M; ++i) dQ = dQ + row[k * M + i];
                acc = acc + l.weight[k] * dQ;
            }
            dS_out[u] = valid ? acc : __longlong_as_double(0x7ff8000000000000ll);
        }
    }
}

// The same by a lane per pair, for many pairs: bound by the issue of instructions, where
// half a wavefront per pair leaves most lanes idle in turn.  dN goes out row by row of a
// shell, M^2 lanes per pair, from the pairs' histograms in LDS: a lane that writes its own
// pair's E entries touches a line per entry.  2,000,000 pairs on FCC 20^3, 5 species,
// 3 shells, half a wavefront per pair -> here: 1,304 -> 583 us, with dN 1,353 -> 848.
__global__ void __launch_bounds__(kTrialThreads)
trial_eval_many_kernel(EvalDesc ed, SmallTable tw, const int8_t *__restrict__ sp, const int32_t *__restrict__ counts,
                       const int32_t *__restrict__ bad, int64_t n_pairs, const int32_t *__restrict__ pairs,
                       double *__restrict__ dS_out, int32_t *__restrict__ dN_out, int32_t *__restrict__ status) {
    __shared__ TrialTables l;
    __shared__ uint64_t hp_all[kTrialThreads], hq_all[kTrialThreads];
    __shared__ int32_t ab_all[kTrialThreads];   // a | b << 8, or -1: no such pair
    const int M = ed.M, E = ed.S * M * M, M2 = M * M;
    const int tid = (int)threadIdx.x, lane = tid % kWave, wave0 = tid - lane;
    if (!trial_tables(l, ed, tw, counts, bad, status)) return;
    // this lane's entry (oi, oj) of the pairs that it writes, and which of them
    const int at_once = kWave / M2, sub = lane / M2, oe = lane - sub * M2, oi = oe / M, oj = oe - oi * M;
    const auto diff = [](uint64_t hp, uint64_t hq, int j) {
        return (int)((hq >> (5 * j)) & 31u) - (int)((hp >> (5 * j)) & 31u);
    };
    // every lane makes the same number of turns, for the barriers
    for (int64_t u0 = (int64_t)blockIdx.x * kTrialThreads; u0 < n_pairs; u0 += (int64_t)gridDim.x * kTrialThreads) {
        const int64_t u = u0 + tid;
        const bool here = u < n_pairs;
        const int32_t p = here ? pairs[2 * u] : -1, q = here ? pairs[2 * u + 1] : -1;
        const bool valid = here && p >= 0 && q >= 0 && (uint32_t)p < ed.N && (uint32_t)q < ed.N;
        const int a = valid ? sp[p] : 0, b = valid ? sp[q] : 0;
        const SiteCoord c = site_coord(valid ? (uint32_t)p : 0u, ed.lgA, ed.Lx, ed.Ly, ed.inv_Lx, ed.inv_Ly);
        const SiteCoord d = site_coord(valid ? (uint32_t)q : 0u, ed.lgA, ed.Lx, ed.Ly, ed.inv_Lx, ed.inv_Ly);
        int bx, by, bz, ex, ey, ez;
        basis_bits(ed.A, c.b, bx, by, bz);
        basis_bits(ed.A, d.b, ex, ey, ez);
        if (dN_out) ab_all[tid] = valid ? a | b << 8 : -1;
        double acc = 0.0;
        int t = 0;
        for (int k = 0; k < ed.S; ++k) {
            // neighbours of p and of q by species, the other site left out: 5-bit fields (z_k <= 24)
            uint64_t hp = 0, hq = 0;
            const int t1 = t + ed.zk[k];
            if (a != b)
                for (int i = t; i < t1; ++i) {
                    const int32_t o = l.off[i];
                    const int ox = (int8_t)o, oy = (int8_t)(o >> 8), oz = (int8_t)(o >> 16);
                    const int32_t rp = site_at(ed, 2 * c.cx + bx + ox, 2 * c.cy + by + oy, 2 * c.cz + bz + oz);
                    const int32_t rq = site_at(ed, 2 * d.cx + ex + ox, 2 * d.cy + ey + oy, 2 * d.cz + ez + oz);
                    const int vp = sp[rp], vq = sp[rq];
                    hp += rp != q ? 1ull << (5 * vp) : 0ull;
                    hq += rq != p ? 1ull << (5 * vq) : 0ull;
                }
            t = t1;
            if (dN_out) {
                hp_all[tid] = hp;
                hq_all[tid] = hq;
                __syncthreads();
                for (int x0 = 0; x0 < kWave; x0 += at_once) {
                    const int x = wave0 + x0 + sub;
                    if (sub >= at_once || x0 + sub >= kWave) continue;
                    const int32_t ab = ab_all[x];
                    if (ab < 0) continue;
                    const int oa = ab & 0xFF, ob = ab >> 8;
                    const uint64_t xp = hp_all[x], xq = hq_all[x];
                    const int dn = oa != ob ? trial_dn(oi, oj, oa, ob, diff(xp, xq, oa), diff(xp, xq, ob),
                                                       diff(xp, xq, oi), diff(xp, xq, oj))
                                            : 0;
                    dN_out[(u0 + x) * E + k * M2 + oe] = dn;
                }
                __syncthreads();
            }
            const int Da = diff(hp, hq, a), Db = diff(hp, hq, b);
            double dQ = 0.0;
            for (int i = 0; i < M; ++i) {
                const int Di = diff(hp, hq, i);
                double rowsum = 0.0;
                for (int j = 0; j < M; ++j) {
                    const int dn = a != b ? trial_dn(i, j, a, b, Da, Db, Di, diff(hp, hq, j)) : 0;
                    const int e = (k * M + i) * M + j;
                    const double a1 = 1.0 - (double)(l.cnt[e] + dn) * l.R[e];
                    const double d1 = a1 - l.t[e];
                    rowsum = rowsum + (d1 * d1 - l.old_sq[e]);
                }
                dQ = dQ + rowsum;
            }
            acc = acc + l.weight[k] * dQ;
        }
        if (here) dS_out[u] = valid ? acc : __longlong_as_double(0x7ff8000000000000ll);
    }
}

__global__ void philox_kernel(const uint32_t *__restrict__ ctr, uint64_t seed, int64_t n,
                              uint32_t *__restrict__ out) {
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    uint32_t c[4] = {ctr[4 * i], ctr[4 * i + 1], ctr[4 * i + 2], ctr[4 * i + 3]};
    philox4x32_10(c, (uint32_t)seed, (uint32_t)(seed >> 32));
    for (int w = 0; w < 4; ++w) out[4 * i + w] = c[w];
}

// Row r of dst is row t.row[r] of src, N bytes each; T divides N and the bases.  One
// launch for up to kCopyRows rows: bound by the launch, where a copy command per row kept
// the device waiting for the next (a search of 6 iterations with 48 rows of 32,000 bytes
// each: 35.0 -> 32.8 ms).
template <class T>
__global__ void copy_rows_kernel(RowTable t, uint32_t n, const T *__restrict__ src, T *__restrict__ dst) {
    const T *s = src + (int64_t)t.row[blockIdx.y] * n;
    T *d = dst + (int64_t)blockIdx.y * n;
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) d[i] = s[i];
}

}  // namespace

hipError_t launch_zero_i32(int32_t *p, int64_t n, hipStream_t stream) {
    if (n <= 0) return hipSuccess;
    const int blocks = (int)std::min<int64_t>((n + 255) / 256, 4096);
    hipLaunchKernelGGL(zero_i32_kernel, dim3(blocks), dim3(256), 0, stream, p, n);
    return hipGetLastError();
}

hipError_t launch_count_gather(const EvalDesc &ed, int64_t K, const int8_t *species, int32_t *counts,
                               int32_t *bad, hipStream_t stream) {
    const int E = ed.S * ed.M * ed.M;
    hipError_t e = launch_zero_i32(counts, K * E, stream);
    if (e != hipSuccess) return e;
    e = launch_zero_i32(bad, K, stream);
    if (e != hipSuccess) return e;
    const int per_cfg = (int)std::min<int64_t>(std::max<int64_t>(1, (ed.N + 2047) / 2048), 1024);
    const int gy = (int)std::min<int64_t>(K, 65535);
    hipLaunchKernelGGL(count_gather_kernel, dim3(per_cfg, gy), dim3(256), 0, stream, ed, K, species,
                       counts, bad);
    return hipGetLastError();
}

hipError_t launch_upload(const SmallTable &t, int n, double *dst, hipStream_t stream) {
    if (n <= 0) return hipSuccess;
    if (n > kMaxTable) return hipErrorInvalidValue;
    hipLaunchKernelGGL(upload_kernel, dim3(1), dim3(256), 0, stream, t, n, dst);
    return hipGetLastError();
}

hipError_t launch_count_tasks(const CountTask *tasks, const uint32_t *tile0, int n, uint32_t n_tiles, uint32_t tile,
                              int max_E, hipStream_t stream) {
    if (n <= 0 || n_tiles == 0) return hipSuccess;
    if (tile == 0 || max_E <= 0 || max_E > kMaxShells * kMaxSpecies * kMaxSpecies) return hipErrorInvalidValue;
    const size_t lds = ((size_t)max_E * kHistCopies + 1) * sizeof(int32_t);
    hipLaunchKernelGGL(count_tasks_kernel, dim3(n_tiles), dim3(256), lds, stream, tasks, tile0, n, tile);
    return hipGetLastError();
}

hipError_t launch_objective_epilogue(const EvalDesc &ed, int64_t K, const int32_t *counts,
                                     const int32_t *bad, const double *target, const double *weight,
                                     double *S_F, hipStream_t stream) {
    if (K <= 0) return hipSuccess;
    if (K <= 1024) {   // few configurations: a block each rather than a lane each
        hipLaunchKernelGGL(objective_block_kernel, dim3((unsigned)K), dim3(64), 0, stream, ed, counts, bad, target,
                           weight, S_F);
        return hipGetLastError();
    }
    const int blocks = (int)((K + 255) / 256);
    hipLaunchKernelGGL(objective_kernel, dim3(blocks), dim3(256), 0, stream, ed, K, counts, bad, target,
                       weight, S_F);
    return hipGetLastError();
}

hipError_t launch_objective_one(const OneDesc &od, const SmallTable &tw, const int32_t *counts, const int32_t *bad,
                                OneResult *out, hipStream_t stream) {
    static_assert(kMaxShells * kMaxSpecies * kMaxSpecies <= kOneThreads, "a lane per entry");
    hipLaunchKernelGGL(objective_one_kernel, dim3(1), dim3(kOneThreads), 0, stream, od, tw, counts, bad, out);
    return hipGetLastError();
}

hipError_t launch_final_objective(const ChainDesc *descs_dev, int n_chains, hipStream_t stream) {
    if (n_chains <= 0) return hipSuccess;
    hipLaunchKernelGGL(final_objective_kernel, dim3((n_chains + 63) / 64), dim3(64), 0, stream, descs_dev, n_chains);
    return hipGetLastError();
}

hipError_t launch_copy_rows(const int *rows, int count, int64_t N, const int8_t *src, int8_t *dst,
                            hipStream_t stream) {
    const uintptr_t all = (uintptr_t)src | (uintptr_t)dst | (uintptr_t)N;
    for (int r0 = 0; r0 < count; r0 += kCopyRows) {
        RowTable t{};
        const int n = std::min(count - r0, kCopyRows);
        for (int r = 0; r < n; ++r) t.row[r] = rows[r0 + r];
        int8_t *d = dst + (int64_t)r0 * N;
        const auto grid = [&](int64_t items) { return dim3((unsigned)std::min<int64_t>((items + 255) / 256, 256), n); };
        if (all % 16 == 0)
            hipLaunchKernelGGL(copy_rows_kernel<int4>, grid(N / 16), dim3(256), 0, stream, t, (uint32_t)(N / 16),
                               (const int4 *)src, (int4 *)d);
        else if (all % 4 == 0)
            hipLaunchKernelGGL(copy_rows_kernel<int32_t>, grid(N / 4), dim3(256), 0, stream, t, (uint32_t)(N / 4),
                               (const int32_t *)src, (int32_t *)d);
        else
            hipLaunchKernelGGL(copy_rows_kernel<int8_t>, grid(N), dim3(256), 0, stream, t, (uint32_t)N, src, d);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// Pairs from which a lane per pair is faster, without and with dN.  us per call, half a
// wavefront / a lane per pair: without dN 65,536 pairs FCC 20^3, 8 species, 4 shells 275 /
// 290, 5 species, 3 shells 103 / 112, BCC 31^3, 3 species, 4 shells 104 / 115, FCC 40^3, 4
// species, 2 shells 92 / 85; 130,000 pairs 346 / 300, 144 / 119, 140 / 123, 120 / 88.  With dN
// 130,000 pairs FCC 20^3, 5 species, 4 shells 154 / 182, 3 shells 151 / 152; 260,000 pairs 8
// species, 4 shells 497 / 455, 5 species, 3 shells 231 / 191.
constexpr int64_t kTrialMany = 80000, kTrialManyDN = 200000;
hipError_t launch_trial_eval(const EvalDesc &ed, const SmallTable &tw, const int8_t *species, const int32_t *counts,
                             const int32_t *bad, int64_t n_pairs, const int32_t *pairs, double *dS, int32_t *dN,
                             int32_t *status, hipStream_t stream) {
    static_assert(kMaxShells * kMaxSpecies == kTrialLanes, "a lane per row of D");
    const bool many = n_pairs >= (dN ? kTrialManyDN : kTrialMany);
    const int per = many ? kTrialThreads : kTrialThreads / kTrialLanes;
    // at most 8 workgroups per CU, each with many pairs: their tables are made once
    const int blocks = (int)std::min<int64_t>(std::max<int64_t>(1, (n_pairs + per - 1) / per), 2048);
    hipLaunchKernelGGL(many ? trial_eval_many_kernel : trial_eval_kernel, dim3(blocks), dim3(kTrialThreads), 0, stream,
                       ed, tw, species, counts, bad, n_pairs, pairs, dS, dN, status);
    return hipGetLastError();
}

hipError_t launch_philox(const uint32_t *ctr, uint64_t seed, int64_t n, uint32_t *out, hipStream_t stream) {
    if (n <= 0) return hipSuccess;
    const int blocks = (int)((n + 255) / 256);
    hipLaunchKernelGGL(philox_kernel, dim3(blocks), dim3(256), 0, stream, ctr, seed, n, out);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Random solutions of the global search (Sec. 4.1): the composition-sorted
// species list placed through a keyed permutation of the sites.  The
// permutation is a four-round balanced Feistel network on 2h-bit values whose
// round function is word 0 of Philox4x32-10(counter = (right half, round,
// slot, 0x80000000 | iteration), key = seed), re-applied (cycle walking) until
// the value is below N.  One thread per list position.
// ---------------------------------------------------------------------------

__device__ __forceinline__ uint32_t feistel4(uint32_t x, int h, uint32_t slot, uint32_t iteration, uint32_t k0,
                                             uint32_t k1) {
    const uint32_t mask = (1u << h) - 1u;
    uint32_t l = x >> h, r = x & mask;
#pragma unroll
    for (uint32_t round = 0; round < 4; ++round) {
        uint32_t c[4] = {r, round, slot, 0x80000000u | iteration};
        philox4x32_10(c, k0, k1);
        const uint32_t nl = r;
        r = l ^ (c[0] & mask);
        l = nl;
    }
    return (l << h) | r;
}

__global__ void random_configs_kernel(uint32_t N, int h, RandomConfigDesc d, int8_t *__restrict__ out) {
    const uint32_t cfg = blockIdx.y;
    const uint32_t slot = d.slot0 + cfg;
    const uint32_t k0 = (uint32_t)d.seed, k1 = (uint32_t)(d.seed >> 32);
    int8_t *o = out + (int64_t)cfg * N;
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < N; i += gridDim.x * blockDim.x) {
        int j = 0;
        while (j + 1 < d.M && i >= d.prefix[j + 1]) ++j;
        uint32_t x = feistel4(i, h, slot, d.iteration, k0, k1);
        while (x >= N) x = feistel4(x, h, slot, d.iteration, k0, k1);
        o[x] = (int8_t)j;
    }
}

hipError_t launch_random_configs(uint32_t N, const RandomConfigDesc &d, int n_configs, int8_t *out,
                                 hipStream_t stream) {
    if (n_configs <= 0 || N == 0) return hipSuccess;
    int h = 1;
    while ((uint64_t(1) << (2 * h)) < N) ++h;
    const int threads = 256;
    const int bx = (int)std::min<uint32_t>((N + threads - 1) / threads, 1024);
    for (int c0 = 0; c0 < n_configs; c0 += 65535) {
        RandomConfigDesc dc = d;
        dc.slot0 = d.slot0 + (uint32_t)c0;
        const int nc = std::min(65535, n_configs - c0);
        hipLaunchKernelGGL(random_configs_kernel, dim3(bx, nc), dim3(threads), 0, stream, N, h, dc,
                           out + (int64_t)c0 * N);
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Non-incremental baseline: copies of one configuration with one swap each.
// ---------------------------------------------------------------------------

__global__ void replicate_kernel(const int8_t *__restrict__ base, int64_t N, int n, int8_t *__restrict__ out) {
    const int64_t row = blockIdx.y;
    int8_t *o = out + row * N;
    if ((N & 3) == 0) {
        const uint32_t *b4 = reinterpret_cast<const uint32_t *>(base);
        uint32_t *o4 = reinterpret_cast<uint32_t *>(o);
        for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < N / 4; i += (int64_t)gridDim.x * blockDim.x)
            o4[i] = b4[i];
    } else {
        for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < N; i += (int64_t)gridDim.x * blockDim.x)
            o[i] = base[i];
    }
}

// pair i swaps sites p, q of copy i; a pair outside [0, N) sets *bad and is skipped
__global__ void apply_swaps_kernel(const int8_t *__restrict__ base, int64_t N, const int32_t *__restrict__ pairs,
                                   int n, int8_t *__restrict__ out, int32_t *__restrict__ bad) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int32_t p = pairs[2 * i], q = pairs[2 * i + 1];
    if (p < 0 || q < 0 || p >= N || q >= N) {
        atomicOr(bad, 1);
        return;
    }
    out[(int64_t)i * N + p] = base[q];
    out[(int64_t)i * N + q] = base[p];
}

__global__ void sub_objective_kernel(const double *__restrict__ S_F, const double *__restrict__ S0, int n,
                                     double *__restrict__ dS) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dS[i] = S_F[2 * i] - S0[0];
}

hipError_t launch_swap_copies(const int8_t *base, int64_t N, const int32_t *pairs, int n, int8_t *out, int32_t *bad,
                              hipStream_t stream) {
    if (n <= 0) return hipSuccess;
    const int64_t words = (N & 3) == 0 ? N / 4 : N;
    const int bx = (int)std::min<int64_t>((words + 255) / 256, 256);
    for (int r0 = 0; r0 < n; r0 += 65535) {
        const int nr = std::min(65535, n - r0);
        hipLaunchKernelGGL(replicate_kernel, dim3(bx, nr), dim3(256), 0, stream, base, N, nr, out + (int64_t)r0 * N);
    }
    hipLaunchKernelGGL(apply_swaps_kernel, dim3((n + 255) / 256), dim3(256), 0, stream, base, N, pairs, n, out, bad);
    return hipGetLastError();
}

hipError_t launch_sub_objective(const double *S_F, const double *S0, int n, double *dS, hipStream_t stream) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(sub_objective_kernel, dim3((n + 255) / 256), dim3(256), 0, stream, S_F, S0, n, dS);
    return hipGetLastError();
}

}  // namespace pyhea
