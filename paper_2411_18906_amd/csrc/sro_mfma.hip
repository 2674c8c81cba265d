// Full SRO evaluation on the matrix cores (Sec. 4.3, Eq. 2): pair counts as
// contractions of 4-bit features.
//
// A species is a code of three bits, one nibble per site: 1, 2, 4, 6 for species
// 0 .. P - 1 (P = M - 1) and 0 for the last.  Read as a 4-bit float (E2M1), the
// code ANDed with the row mask 1, 2, 4 or 6 gives four features of the site,
//    f = {1/2 a0, a1 + a3, 2 (a2 + a3), a1 + 2 a2 + 4 a3},  a_i = [species = i],
// which determine a0 .. a3, so sums of feature products over pairs of sites
// determine the pair counts.  A matrix instruction of 16 rows (sublattice and
// feature at a cell), 16 columns (sublattice and feature at the displaced cell)
// and 128 cells adds the products of one displacement: products are at most 16 and
// multiples of 1/4, and a wavefront counts at most kMfmaMaxCells cells, so every
// binary32 sum is exact.
//
// Layout: word q of a column (x, y) and a sublattice holds layers W p + q - dead in its
// nibbles p, so a layer up or down is the neighbouring word; the word above the last is the
// first shifted by a nibble, the one below the first is held as one word more.  The dead
// slots below layer 0 (fewer than W) repeat the last layers, and are masked in the centre.
// The four words of a 16-byte fragment, what a lane
// gives to a matrix instruction (its 32 cells), are word q of the columns x, x + xs,
// x + 2 xs and x + 3 xs: the row's quarters, so a column left or right is the neighbouring
// fragment (at a quarter's end a copy with its words rotated).  The four 16-lane groups of
// a wavefront take four rows.  A wavefront walks x and holds fragments x - 1, x, x + 1 of
// the row above and x, x + 1 of its own in registers: a step of 128 cells reads four
// fragments from LDS (these two's next, the layers below and above) for all its
// displacements, and shifts or moves no word.
//
// Displacements are one of each +-d pair of cells: (0, 0, dz = 0, 1), (1, 0, dz)
// and (dx, 1, dz) with dx, dz in -1, 0, 1; +-1 in z is the centre's fragment below or
// above.  FCC has 4 sublattices x 4 features.  BCC has 2; its rows also hold the centre's
// layer below, its columns the row above, so 6 instructions cover all displacements.
// Which sublattice pairs of a displacement belong to which shell is a list of
// the host; the site's products with itself give the species totals.
//
// What bounds it: the issue of instructions.  FCC 20^3, 5 species, 3 shells, per wavefront:
// 4,200 cycles of matrix instructions and about 1,300 vector instructions of 4 cycles
// (conversion 250, masks and addresses of the steps 500, starts of rows 180, sums 120), of
// about 10,000 cycles; the conversion's reads and the end of Eq. 2-3 overlap with the other
// three workgroups of the CU.  32,768 such configurations (1.05 GB read once, 0.21 ms as a
// copy goes): 0.57 ms; bit-sliced 0.83.  FCC 40^3, 4 species, 2 shells, 4,096: 0.38 / 0.43 ms;
// BCC 31^3, 5 species, 3 shells, 2,048: 0.088 / 0.138 ms.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <mutex>
#include <set>
#include <type_traits>
#include <vector>

#include "device_common.h"
#include "mc_kernels.h"
#include "sro_mfma.h"

namespace pyhea {

namespace {

using v4i = int __attribute__((ext_vector_type(4)));
using v8i = int __attribute__((ext_vector_type(8)));
using v4f = float __attribute__((ext_vector_type(4)));

// a float whose last bit is 1/4: its bits count the quarters added to it.  Integers because
// the LDS adds floats at a lane per 3 cycles (five times the whole kernel's time).
constexpr float kQuarter = 1.5f * (1 << 21);

__device__ __forceinline__ v4f mfma4(v4i a, v4i b, v4f c) {
    // both operands 4-bit floats (format 4), four registers each; no block scales
    const v8i a8 = __builtin_shufflevector(a, a, 0, 1, 2, 3, -1, -1, -1, -1);
    const v8i b8 = __builtin_shufflevector(b, b, 0, 1, 2, 3, -1, -1, -1, -1);
    return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(a8, b8, c, 4, 4, 0, 0, 0, 0);
}

__device__ __forceinline__ uint32_t perm(uint32_t hi, uint32_t lo, uint32_t sel) {
    return __builtin_amdgcn_perm(hi, lo, sel);
}

// Counts and Eq. 2-3 of one configuration from its feature sums F [groups][4][4]
// (units of 1/4; group S: sites with themselves) and the invalid-id flag.
template <class Sum>
struct FinishLds {
    Sum G[kMfmaGroups][16];
    int32_t n[8];
    int32_t lc[kMaxShells * 25];
    double lsq[kMaxShells * 25];
    double lrow[kMaxShells * 5];
};
constexpr int kFinishThreads = 128;   // S M^2 <= 100 entries at once: 6,500 clocks, 11,000 by one wavefront
// The whole workgroup calls it, for its barriers; the first two wavefronts do the work.
template <class Sum>
__device__ __forceinline__ void finish(const Sum *F, bool bad, const MfmaDesc &md, FinishLds<Sum> &l, int32_t *cnt,
                                       int32_t *bad_out, const double *tw, double *S_F) {
    const int M = md.M, S = md.S, P = M - 1;
    const int tid = (int)threadIdx.x;
    const int g = tid >> 2, u = tid & 3;
    // rows of features to species, then columns: the sums by species pairs
    if (g <= S) {
        Sum a[4];
        species_of_features(F[g * 16 + u], F[g * 16 + 4 + u], F[g * 16 + 8 + u], F[g * 16 + 12 + u], a);
        for (int i = 0; i < 4; ++i) l.G[g][4 * i + u] = a[i];
    }
    __syncthreads();
    if (g <= S) {
        Sum a[4];
        species_of_features(l.G[g][4 * u], l.G[g][4 * u + 1], l.G[g][4 * u + 2], l.G[g][4 * u + 3], a);
        for (int j = 0; j < 4; ++j) l.G[g][4 * u + j] = a[j];
        if (g == S) l.n[u] = (int32_t)(u == 0 ? a[0] : u == 1 ? a[1] : u == 2 ? a[2] : a[3]);
    }
    __syncthreads();
    const int32_t n_last = (int32_t)md.N - l.n[0] - l.n[1] - l.n[2] - l.n[3];   // (species beyond P are 0)
    // N_ij = H_ij + H_ji (one of each +-d pair was counted); the last species from the rows' sums
    if (g < S) {
        int32_t *c = l.lc + g * M * M;
        int32_t r = md.zk[g] * l.n[u];   // (modulo 2^32; the counts themselves fit)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int32_t v = (int32_t)(l.G[g][4 * u + j] + l.G[g][4 * j + u]);
            r -= v;   // (0 beyond P)
            if (u < P && j < P) c[u * M + j] = v;
        }
        if (u < P) {
            c[u * M + P] = r;
            c[P * M + u] = r;
        }
        int32_t all = r;   // over the quad
        all += __builtin_amdgcn_update_dpp(0, all, 0xB1, 0xF, 0xF, true);   // quad_perm 1,0,3,2
        all += __builtin_amdgcn_update_dpp(0, all, 0x4E, 0xF, 0xF, true);   // quad_perm 2,3,0,1
        if (u == 0) c[P * M + P] = md.zk[g] * n_last - all;
    }
    if (tid == 0) {
        *bad_out = bad ? 1 : 0;
        l.n[P] = n_last;   // (read above by every lane of this wavefront, and P < 4 there holds 0 besides)
    }
    __syncthreads();
    if (tid < S * M * M) {
        const int e = tid;
        cnt[e] = l.lc[e];
        if (S_F) {
            const int row = e * (65536 / M + 1) >> 16, k = row * (65536 / M + 1) >> 16;
            const int64_t ni = l.n[row - k * M], nj = l.n[e - row * M];
            const double R = (double)md.N / (double)(ni * nj * (int64_t)md.zk[k]);
            const double a = 1.0 - (double)l.lc[e] * R;
            const double dd = a - tw[e];
            l.lsq[e] = dd * dd;
        }
    }
    if (!S_F) return;
    __syncthreads();
    if (tid < S * M) {
        double row = 0.0;
        for (int j = 0; j < M; ++j) row = row + l.lsq[tid * M + j];
        l.lrow[tid] = row;
    }
    __syncthreads();
    if (tid == 0) {
        bool ok = !bad;
        for (int i = 0; i < M; ++i) ok = ok && l.n[i] > 0;
        double sum = 0.0;
        for (int k = 0; k < S; ++k) {
            double Q = 0.0;
            for (int i = 0; i < M; ++i) Q = Q + l.lrow[k * M + i];
            sum = sum + tw[S * M * M + k] * Q;
        }
        const double nan = __longlong_as_double(0x7ff8000000000000ll);
        S_F[0] = ok ? sum : nan;
        S_F[1] = ok ? sqrt(sum) : nan;
    }
}

struct Shared {
    MfmaGroupSum F[kMfmaGroups * 16];
    int32_t bad;
    uint8_t list[kMfmaTiles * 16];
    FinishLds<MfmaGroupSum> fin;
};
constexpr int kFixedLds = (int)((sizeof(Shared) + 15) & ~size_t(15));

__device__ __forceinline__ v4i masked(v4i v, uint32_t m) {
    return v4i{v[0] & (int)m, v[1] & (int)m, v[2] & (int)m, v[3] & (int)m};
}

// A lane's fragments in LDS at x = 0: its centre and its columns of the row above (BCC:
// its columns), the words below and above, and the word of layer 0.
struct Rows {
    const v4i *p0, *p1, *pm, *pp, *pf;
};
struct Masks {
    uint32_t feature, centre;   // the centre's without dead slots; 0 in rows past the last
    int up;
};

// What a step carries to the next; its three uses are rotated by name, not moved.
template <int kT, bool kQ, int kU>
__device__ __forceinline__ void count_step(v4f (&acc)[kT], const Rows &r, const Masks &k, int x, int xs, int Lx,
                                           bool last, int top, v4i &c0, v4i &c1, v4i &cn, v4i &wm, v4i &wc, v4i &wp) {
    constexpr bool fcc = kT != 6;
    v4i am = r.pm[kU], ap = r.pp[kU];   // site z holds the code of z - 1 / z + 1
    v4i n0;
    // the fragments of the next step's x + 1 (unused after the last column)
    if constexpr (fcc) n0 = r.p0[kU + 2];
    const v4i n1 = r.p1[kU + 2];
    v4i a0 = c0;
    uint32_t m[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        m[j] = kQ ? k.centre : j * xs + x < Lx ? k.centre : 0u;   // columns past the row's end
        if constexpr (fcc) a0[j] &= (int)m[j];
        am[j] &= (int)m[j];
    }
    // tiles in the order of mfma_tiles()
    if constexpr (!fcc) {
        acc[0] = mfma4(am, wm, acc[0]);
        acc[1] = mfma4(am, wc, acc[1]);
        acc[2] = mfma4(am, wp, acc[2]);
    } else {
        acc[0] = mfma4(a0, c0, acc[0]);
        acc[2] = mfma4(a0, c1, acc[2]);
        acc[5] = mfma4(a0, wm, acc[5]);
        acc[6] = mfma4(a0, wc, acc[6]);
        acc[7] = mfma4(a0, wp, acc[7]);
        acc[1] = mfma4(am, c0, acc[1]);
        acc[3] = mfma4(am, c1, acc[3]);
        acc[8] = mfma4(am, wc, acc[8]);
        if constexpr (kT == 14) {
            acc[10] = mfma4(am, wm, acc[10]);
            acc[11] = mfma4(am, wp, acc[11]);
        }
    }
    if (last) {   // uniform; a loop of its own would cost more registers than there are
        const v4i ef = r.pf[kU];
#pragma unroll
        for (int j = 0; j < 4; ++j) ap[j] = (int)(((uint32_t)ap[j] >> 4) | (((uint32_t)ef[j] & 0xFu) << top));
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) ap[j] &= (int)(fcc || !k.up ? m[j] : 0u);
    if constexpr (!fcc) {
        acc[3] = mfma4(ap, wm, acc[3]);
        acc[4] = mfma4(ap, wc, acc[4]);
        acc[5] = mfma4(ap, wp, acc[5]);
    } else {
        acc[4] = mfma4(ap, c1, acc[4]);
        acc[9] = mfma4(ap, wc, acc[9]);
        if constexpr (kT == 14) {
            acc[12] = mfma4(ap, wm, acc[12]);
            acc[13] = mfma4(ap, wp, acc[13]);
        }
        cn = masked(n0, k.feature);
    }
    wm = masked(n1, k.feature);
}

// Columns x .. x1 - 1 of a word of four rows (r at x).  last: word W - 1, whose upper
// neighbour is word 0 shifted.
template <int kT, bool kQ>
__device__ __forceinline__ void walk(v4f (&acc)[kT], Rows r, const Masks &k, int x, int x1, int xs, int Lx, bool last,
                                     int top) {
    v4i a0, a1, a2, b0 = masked(r.p1[-1], k.feature), b1 = masked(r.p1[0], k.feature), b2 = masked(r.p1[1], k.feature);
    if constexpr (kT != 6) {
        a0 = masked(r.p0[0], k.feature);
        a1 = masked(r.p0[1], k.feature);
    }
    while (true) {
        count_step<kT, kQ, 0>(acc, r, k, x, xs, Lx, last, top, a0, a1, a2, b0, b1, b2);
        if (++x == x1) break;
        count_step<kT, kQ, 1>(acc, r, k, x, xs, Lx, last, top, a1, a2, a0, b1, b2, b0);
        if (++x == x1) break;
        count_step<kT, kQ, 2>(acc, r, k, x, xs, Lx, last, top, a2, a0, a1, b2, b0, b1);
        if (++x == x1) break;
        r.p0 += 3;
        r.p1 += 3;
        r.pm += 3;
        r.pp += 3;
        r.pf += 3;
    }
}

// kT: displacement tiles (14 or 10: FCC; 6: BCC); kQ: Lx and every workgroup's rows are multiples of 4
template <int kT, bool kQ>
__global__ void __launch_bounds__(512, 4)
count_mfma_kernel(MfmaDesc md, int64_t K, const int8_t *__restrict__ species, int32_t *__restrict__ partial,
                  int32_t *__restrict__ counts, int32_t *__restrict__ bad_out, const double *__restrict__ tw,
                  double *__restrict__ S_F) {
    constexpr int A = kT == 6 ? 2 : 4;
    typedef std::conditional_t<A == 4, uint32_t, uint16_t> Cell __attribute__((aligned(1), may_alias));
    extern __shared__ __align__(16) uint8_t smem[];
    Shared &sh = *reinterpret_cast<Shared *>(smem);
    v4i *D = reinterpret_cast<v4i *>(smem + kFixedLds);           // [R] rows of [W + 1][A][Xs]: words -1 .. W - 1, x = -1 .. xs
    int32_t *T = reinterpret_cast<int32_t *>(D);                  // then [kT][4][64]: sums by tile, in quarters
    // a configuration's workgroups on one XCD (block b runs on XCD b mod 8): they share their border rows in its L2
    const uint32_t nc = (uint32_t)md.nchunks;
    const int64_t kc = nc == 1 ? blockIdx.x : (int64_t)(blockIdx.x / (8 * nc)) * 8 + blockIdx.x % 8;
    const int chunk = nc == 1 ? 0 : (int)((blockIdx.x / 8) % nc);
    if (kc >= K) return;
    const int tid = (int)threadIdx.x, nthreads = (int)blockDim.x;
    const int Lx = md.Lx, Ly = md.Ly, W = md.W, xs = md.xs, Xs = md.Xs, RS = md.RS;
    const int y0 = chunk * md.ys;
    const int ny = min(md.ys, Ly - y0);            // centre rows
    const int R = min(md.R, ny + 1);               // rows held (all of them wrap around by themselves)
    if (tid < kMfmaGroups * 16) sh.F[tid] = 0;
    if (tid == 0) sh.bad = 0;
    for (int i = tid; i < kT * 4; i += nthreads)
        reinterpret_cast<uint32_t *>(sh.list)[i] = reinterpret_cast<const uint32_t *>(md.list)[i];

    bool bad = false;
    // ---- 1. codes: a lane makes the fragments of an (x, row, q), all sublattices ----------
    {
        const uint8_t *cfg = reinterpret_cast<const uint8_t *>(species) + kc * (int64_t)md.N;
        const uint32_t layer = (uint32_t)(Lx * Ly) * A;
        const uint32_t last = (uint32_t)(md.M - 1) * 0x01010101u;   // nibbles past the last: the species of code 0
        const double inv_xs = md.inv_xs, inv_R = R == md.R ? md.inv_R : 1.0 / (double)R;
        uint32_t bad_id = 0, bad_code = 0;
        const int top = 4 * (md.NP - 1);
        const uint32_t codes_hi = md.codes_hi;
        uint32_t codes_lo = md.codes_lo;
        asm volatile("" : "+v"(codes_lo));   // (an instruction takes one scalar operand)
#pragma unroll 1
        for (int c = tid; c < R * W * xs; c += nthreads) {
            const int rq = (int)div_small((uint32_t)c, inv_xs), x = c - (int)__umul24((uint32_t)rq, (uint32_t)xs);
            const int q = (int)div_small((uint32_t)rq, inv_R), r = rq - (int)__umul24((uint32_t)q, (uint32_t)R);
            const int y = y0 + r >= Ly ? y0 + r - Ly : y0 + r;
            const uint32_t z0 = (uint32_t)(q < md.dead ? q - md.dead + md.Lz : q - md.dead) * layer;
            const uint32_t line = __umul24((uint32_t)y, (uint32_t)Lx) * A, zq = (uint32_t)q * layer;
            uint32_t off[4];
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                int col = s * xs + x;
                if constexpr (!kQ) {
                    if (col >= Lx) col = col - Lx < Lx ? col - Lx : col % Lx;
                }
                off[s] = line + (uint32_t)col * A;
            }
            uint32_t raw[4][8];   // (only NP of the 8 are set and read)
#pragma unroll
            for (int p = 0; p < 8; ++p) {
                if (p >= md.NP) continue;   // uniform
                // a uniform base, so that the loads need no address arithmetic
                uint64_t at = (uint64_t)cfg + (uint64_t)(uint32_t)(p == 0 ? 0 : W * p - md.dead) * layer;
                asm volatile("" : "+s"(at));
                const auto *base = (const __attribute__((address_space(1))) uint8_t *)at;
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    // one load of a cell, on any address
                    const uint32_t o = off[s] + (p == 0 ? z0 : zq);
                    raw[s][p] = *(const __attribute__((address_space(1))) Cell *)(base + o);
                }
            }
            uint32_t e[4][4];   // byte b: nibbles 2 m, 2 m + 1 of sublattice b
            auto pair = [&](uint32_t r0, uint32_t r1) -> uint32_t {
                if constexpr (A == 4) {
                    bad_id |= r0 | r1;
                    return perm(codes_hi, codes_lo, r0) | (perm(codes_hi, codes_lo, r1) << 4);
                } else {
                    const uint32_t two = perm(r1, r0, 0x05040100u), cd = perm(codes_hi, codes_lo, two);
                    bad_id |= two;
                    return cd | (cd >> 12);
                }
            };
#pragma unroll
            for (int m = 0; m < 4; ++m) {   // uniform branches
                if (2 * m + 1 < md.NP) {
#pragma unroll
                    for (int s = 0; s < 4; ++s) e[s][m] = pair(raw[s][2 * m], raw[s][2 * m + 1]);
                } else if (2 * m < md.NP) {
#pragma unroll
                    for (int s = 0; s < 4; ++s) e[s][m] = pair(raw[s][2 * m], last);
                } else {
#pragma unroll
                    for (int s = 0; s < 4; ++s) e[s][m] = 0;
                }
            }
            v4i w[A];
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const uint32_t u0 = perm(e[s][1], e[s][0], 0x05010400u), v0 = perm(e[s][3], e[s][2], 0x05010400u);
                w[0][s] = (int)perm(v0, u0, 0x05040100u);
                w[1][s] = (int)perm(v0, u0, 0x07060302u);
                bad_code |= (uint32_t)w[0][s] | (uint32_t)w[1][s];
                if constexpr (A == 4) {
                    const uint32_t u1 = perm(e[s][1], e[s][0], 0x07030602u), v1 = perm(e[s][3], e[s][2], 0x07030602u);
                    w[A - 2][s] = (int)perm(v1, u1, 0x05040100u);
                    w[A - 1][s] = (int)perm(v1, u1, 0x07060302u);
                    bad_code |= (uint32_t)w[A - 2][s] | (uint32_t)w[A - 1][s];
                }
            }
            v4i *d = D + (int)__umul24((uint32_t)r, (uint32_t)RS) + (int)__umul24((uint32_t)(q + 1), (uint32_t)(A * Xs)) + 1;
#pragma unroll
            for (int b = 0; b < A; ++b) d[b * Xs + x] = w[b];
            if constexpr (kQ) {
                if (x == 0) {
#pragma unroll
                    for (int b = 0; b < A; ++b) d[b * Xs + xs] = v4i{w[b][1], w[b][2], w[b][3], w[b][0]};
                }
                if (x == xs - 1) {
#pragma unroll
                    for (int b = 0; b < A; ++b) d[b * Xs - 1] = v4i{w[b][3], w[b][0], w[b][1], w[b][2]};
                }
            }
            if (q == W - 1) {   // below word 0 (the last layer below layer 0, if that is in it)
                d -= W * A * Xs;
#pragma unroll
                for (int b = 0; b < A; ++b) {
                    v4i v;
#pragma unroll
                    for (int s = 0; s < 4; ++s)
                        v[s] = (int)(((uint32_t)w[b][s] << 4) | (((uint32_t)w[b][s] >> top) & 0xFu));
                    d[b * Xs + x] = v;
                }
            }
        }
        bad = (bad_id & 0xF8F8F8F8u) != 0 || (bad_code & 0x88888888u) != 0;
    }
    __syncthreads();
    if (bad) sh.bad = 1;   // after the barrier: thread 0 has cleared it by then (read after further ones)
    if constexpr (!kQ) {   // the columns beside the quarters
        const uint32_t *Dw = reinterpret_cast<const uint32_t *>(D);
        for (int i = tid; i < R * W * A * 2; i += nthreads) {
            const int x = i & 1 ? xs : -1, r = (i >> 1) / (W * A), qb = (i >> 1) - r * (W * A);
            const int at = r * RS + (A + qb) * Xs + 1;
            v4i w;
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const int col = (s * xs + x + Lx) % Lx, quarter = col / xs;
                w[s] = (int)Dw[(at + col - quarter * xs) * 4 + quarter];
            }
            D[at + x] = w;
        }
        __syncthreads();
    }

    // ---- 2. counting -------------------------------------------------------------------
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), nw = nthreads >> 6;
    const int row = lane & 15, feature = row & 3;
    const int b = A == 4 ? row >> 2 : row >> 3;
    const int up = A == 4 ? 0 : (row >> 2) & 1;   // BCC: columns of the row above / the centre's layer below
    const uint32_t fmask = feature == 3 ? 0x66666666u : 0x11111111u << feature;
    v4f acc[kT];
#pragma unroll
    for (int t = 0; t < kT; ++t) acc[t] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
    const int top = 4 * (md.NP - 1), dead = md.dead;
    const uint32_t used = md.NP == 8 ? fmask : fmask & ((1u << (4 * md.NP)) - 1);
    const int quads = (ny + 3) >> 2, qs = A * Xs;   // fragments from a word to the next
    const v4i *const lane0 = D + (lane >> 4) * RS + (A + b) * Xs + 1;
    // the wavefronts' shares of the steps (4 rows, q, x), in that order: each gets its part of last words
    const int units = quads * W * (md.whole ? 1 : xs), unit = md.whole ? xs : 1;
    int step = units * wave / nw * unit;
    const int end = units * (wave + 1) / nw * unit;
    int q = (int)__builtin_amdgcn_readfirstlane((int)div_small((uint32_t)step, md.inv_xs)), quad = 0;
    int x = step - q * xs;
    while (q >= W) q -= W, ++quad;
#pragma unroll 1
    while (step < end) {
        int y = quad * 4 + (lane >> 4);
        const v4i *rowp = lane0 + quad * 4 * RS + x;
        Masks masks{fmask, q < dead ? used & ~0xFu : used, up};
        if constexpr (!kQ) {
            if (y >= ny) {
                rowp -= y * RS;
                y = 0;
                masks.centre = 0;
            }
        }
        Rows rows;
        rows.p0 = rowp + q * qs;
        rows.p1 = rows.p0;
        if (A == 4 || up) rows.p1 += y + 1 >= R ? -y * RS : RS;
        rows.pm = A == 4 || up ? rows.p0 - qs : rows.p0;   // BCC: the lane's first centre
        rows.pp = q + 1 < W ? rows.p0 + qs : rowp;
        rows.pf = rowp + dead * qs;
        const int x1 = min(xs, x + end - step);
        walk<kT, kQ>(acc, rows, masks, x, x1, xs, Lx, q == W - 1, top);
        step += x1 - x;
        x = 0;
        if (++q == W) q = 0, ++quad;
    }

    // ---- 3. sums by tile over the wavefronts, then by shell ---------------------------------
    __syncthreads();
    for (int i = tid; i < kT * 64; i += nthreads) D[i] = v4i{0, 0, 0, 0};
    __syncthreads();
#pragma unroll
    for (int t = 0; t < kT; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v)
            atomicAdd(T + t * 256 + v * 64 + lane, __float_as_int(acc[t][v] + kQuarter));
    __syncthreads();
    {
        constexpr int kOut = kMfmaGroups * 16;
        const int part = tid / kOut, parts = nthreads / kOut, o = tid - part * kOut;
        const int g = o >> 4, i = (o >> 2) & 3, j = o & 3;
        if (part < parts && g <= md.S) {
            uint32_t sum = 0;
            const uint32_t none = (uint32_t)nw * (uint32_t)__float_as_int(kQuarter);   // (modulo 2^32)
            for (int e = md.start[g] + part; e < md.start[g + 1]; e += parts) {
                const int l = sh.list[e];
                sum += (uint32_t)T[(l >> 4) * 256 + i * 64 + (l & 15) * 4 + j] - none;
            }
            atomicAdd(&sh.F[o], (int)sum);
        }
    }
    __syncthreads();
    if (nc > 1) {
        int32_t *out = partial + (kc * nc + chunk) * kMfmaPartial;
        for (int i = tid; i < kMfmaGroups * 16; i += nthreads) out[i] = sh.F[i];
        if (tid == 0) out[kMfmaGroups * 16] = sh.bad;
        return;
    }
    const int E = md.S * md.M * md.M;
    finish(sh.F, sh.bad != 0, md, sh.fin, counts + kc * (int64_t)E, bad_out + kc, tw, S_F ? S_F + 2 * kc : nullptr);
}

// Workgroup sums -> counts, and Eq. 2-3 when S_F is given: a block per configuration.
// Bound by the latency of the sums' loads: up to 511 workgroups of a large cell are summed by
// six groups of threads, eight loads in flight each (one load after the other: an evaluation of FCC 60 x 511 x 60 took 215 us, now 116).
constexpr int kFinalThreads = 512;   // of cells in more than kFinalFew workgroups; kFinishThreads else
constexpr int kFinalFew = 16;
__global__ void __launch_bounds__(kFinalThreads) finalize_mfma_kernel(MfmaDesc md, const int32_t *__restrict__ partial,
                                                           int32_t *__restrict__ counts, int32_t *__restrict__ bad,
                                                           const double *__restrict__ tw, double *__restrict__ S_F) {
    __shared__ MfmaSum F[kMfmaGroups * 16 + 1];
    __shared__ FinishLds<MfmaSum> fin;
    constexpr int kOut = kMfmaGroups * 16 + 1;
    const int64_t kc = blockIdx.x;
    const int32_t *p = partial + kc * md.nchunks * (int64_t)kMfmaPartial;
    const int tid = (int)threadIdx.x, part = tid / kOut, parts = (int)blockDim.x / kOut, i = tid - part * kOut;
    if (tid < kOut) F[tid] = 0;
    __syncthreads();
    if (part < parts) {
        MfmaSum v = 0;
#pragma unroll 8
        for (int c = part; c < md.nchunks; c += parts) v += p[c * kMfmaPartial + i];   // the flags add up to > 0
        atomicAdd((unsigned long long *)&F[i], (unsigned long long)v);
    }
    __syncthreads();
    const int E = md.S * md.M * md.M;
    finish(F, F[kMfmaGroups * 16] != 0, md, fin, counts + kc * (int64_t)E, bad + kc, tw, S_F ? S_F + 2 * kc : nullptr);
}

// One tile: columns displaced by dx, for each row class (sublattice; BCC:
// sublattice and shift) its layer displacement (2: no centre) and for each
// column class its row displacement.
struct Tile {
    int dx;
    int dz[4];
    int dy[4];
    int b[4], bt[4];   // sublattices of the row and column classes
};

std::vector<Tile> mfma_tiles(int lattice, bool body) {
    std::vector<Tile> out;
    if (lattice == PYHEA_FCC) {
        auto add = [&](int dx, int dy, int dz) {
            Tile t{};
            t.dx = dx;
            for (int q = 0; q < 4; ++q) {
                t.dz[q] = dz;
                t.dy[q] = dy;
                t.b[q] = t.bt[q] = q;
            }
            out.push_back(t);
        };
        add(0, 0, 0);
        add(0, 0, 1);
        add(1, 0, 0);
        add(1, 0, 1);
        add(1, 0, -1);
        add(-1, 1, 0);
        add(0, 1, 0);
        add(1, 1, 0);
        add(0, 1, 1);
        add(0, 1, -1);
        if (body) {
            add(-1, 1, 1);
            add(1, 1, 1);
            add(-1, 1, -1);
            add(1, 1, -1);
        }
        return out;
    }
    for (int op = 0; op < 2; ++op)
        for (int dx = -1; dx <= 1; ++dx) {
            Tile t{};
            t.dx = dx;
            for (int q = 0; q < 4; ++q) {
                const int second = q & 1;
                t.b[q] = t.bt[q] = q >> 1;
                t.dy[q] = second;
                t.dz[q] = op == 0 ? (second ? 1 : 0) : (second ? 2 : -1);
            }
            out.push_back(t);
        }
    return out;
}

}  // namespace

namespace {
// Which class of which tile belongs to which shell: entries 16 * tile + 4 * row class +
// column class, by group (the shells, then the sites with themselves).
struct TileList {
    int tiles = 0;   // 0: not covered
    uint8_t list[kMfmaTiles * 16];
    uint8_t start[kMfmaGroups + 1];
};

// Every pair of sites within the first S shells once, as one of its two directions, in
// the first tile and class that holds it.
TileList make_tile_list(const Geometry &g) {
    TileList out;
    for (int body = 0; body < 2; ++body) {
        const std::vector<Tile> tiles = mfma_tiles(g.lattice, body != 0);
        std::vector<uint8_t> by_group[kMfmaGroups];
        std::set<std::vector<int>> seen;
        int pairs = 0;
        for (size_t t = 0; t < tiles.size(); ++t)
            for (int rc = 0; rc < 4; ++rc)
                for (int cc = 0; cc < 4; ++cc) {
                    const Tile &T = tiles[t];
                    if (T.dz[rc] == 2) continue;
                    int vb[3], vt[3];
                    basis_vector(g.lattice, T.b[rc], vb);
                    basis_vector(g.lattice, T.bt[cc], vt);
                    const int cell[3] = {T.dx, T.dy[cc], T.dz[rc]};
                    int r2 = 0;
                    std::vector<int> fwd = {T.b[rc], T.bt[cc]}, rev = {T.bt[cc], T.b[rc]};
                    for (int a = 0; a < 3; ++a) {
                        const int d = 2 * cell[a] + vt[a] - vb[a];
                        r2 += d * d;
                        fwd.push_back(d);
                        rev.push_back(-d);
                    }
                    int group = kMfmaGroups;
                    if (r2 == 0) group = g.S;
                    for (int k = 0; k < g.S; ++k)
                        if (r2 == g.r2[k]) group = k;
                    if (group == kMfmaGroups || seen.count(fwd) || seen.count(rev)) continue;
                    seen.insert(fwd);
                    by_group[group].push_back((uint8_t)(16 * t + 4 * rc + cc));
                    if (group < g.S) ++pairs;
                }
        if (2 * pairs == g.A * g.Z) {   // all of them
            int n = 0;
            for (int k = 0; k < kMfmaGroups; ++k) {
                out.start[k] = (uint8_t)n;
                for (uint8_t e : by_group[k]) out.list[n++] = e;
            }
            out.start[kMfmaGroups] = (uint8_t)n;
            out.tiles = (int)tiles.size();
            return out;
        }
        if (g.lattice == PYHEA_BCC) break;
    }
    return out;
}

// The lists depend on the lattice and the number of shells alone: made once each.
const TileList &tile_list(const Geometry &g) {
    static std::once_flag made[2][kMaxShells + 1];
    static TileList lists[2][kMaxShells + 1];
    const int l = g.lattice == PYHEA_FCC ? 0 : 1;
    std::call_once(made[l][g.S], [&] { lists[l][g.S] = make_tile_list(g); });
    return lists[l][g.S];
}

// Fragments of a row in LDS: a sublattice's on an odd stride and a row's on 4 modulo 16
// or 12, so the 16 that a wavefront reads at once lie in different banks.
int row_fragments(int W, int A, int xs, int *Xs) {
    *Xs = (xs + 2) | 1;
    int RS = (W + 1) * A * *Xs;
    while (RS % 8 != 4) ++RS;
    return RS;
}
}  // namespace

// Where the matrix cores are the faster way, by what the bit-sliced counting costs there
// (its work grows with species and shells; here only the tiles do), both measured on
// about 2.5e8 sites (bit-sliced / matrix cores, us):
//   FCC, 3-4 shells: 4 species 20^3 172 / 144, 40^3 181 / 127, 5 species 20^3 215 / 149,
//     40^3 224 / 129; 3 species 20^3 130 / 145, 28^3 116 / 150, but 40^3 137 / 126, 48^3 267 / 206.
//   FCC, 2 shells: 5 species 20^3 141 / 131, 12^3 334 / 289; 4 species 20^3 110 / 129,
//     28^3 103 / 130, but 8^3 1040 / 758, 32^3 132 / 112, 40^3 127 / 113.
//   FCC, 1 shell: 5 species 20^3 118 / 128, 8^3 924 / 754, 40^3 130 / 111; 4 species alike.
//   BCC: 4 species, 2 shells 16^3 137 / 128, 24^3 90 / 82, 31^3 115 / 99, but 48^3 94 / 112;
//     3 shells 48^3 119 / 106; 3 species 16^3 116 / 125, 24^3 62 / 82, 48^3 84 / 111.
// (Above 128,000 sites the bit-sliced words no longer fit the LDS several times.)
bool mfma_is_faster(const Geometry &g) {
    const bool small = g.N <= 2048, large = g.N >= 131072;
    if (g.lattice == PYHEA_BCC) return g.M >= 4 && (g.S >= 3 || g.N <= 65536);
    if (g.M <= 3) return g.S >= 3 && large;
    if (g.S >= 3 || (g.S == 2 && g.M == 5)) return true;
    return small || large;
}

bool fill_mfma_desc(const Geometry &g, int lds_budget, int64_t K, MfmaDesc *md) {
    if (K < 1 || g.M > 5 || !mfma_is_faster(g)) return false;
    const TileList &tl = tile_list(g);
    if (tl.tiles == 0) return false;
    std::memset(md, 0, sizeof(*md));
    md->Lx = g.L[0];
    md->Ly = g.L[1];
    md->Lz = g.L[2];
    md->M = g.M;
    md->S = g.S;
    md->N = (uint32_t)g.N;
    for (int k = 0; k < kMaxShells; ++k) md->zk[k] = k < g.S ? g.z[k] : 0;
    const uint8_t code[4] = {1, 2, 4, 6};
    uint8_t tab8[8];
    for (int s = 0; s < 8; ++s) tab8[s] = s < g.M - 1 ? code[s] : s == g.M - 1 ? 0 : 0x8;
    std::memcpy(&md->codes_lo, tab8, 4);
    std::memcpy(&md->codes_hi, tab8 + 4, 4);
    md->tiles = tl.tiles;
    std::memcpy(md->list, tl.list, sizeof(md->list));
    std::memcpy(md->start, tl.start, sizeof(md->start));

    md->W = (g.L[2] + 7) / 8;   // 8 layers per word
    md->NP = (g.L[2] + md->W - 1) / md->W;
    md->dead = md->W * md->NP - g.L[2];
    md->xs = (g.L[0] + 3) / 4;
    md->RS = row_fragments(md->W, g.A, md->xs, &md->Xs);
    // (the step past a row's last column reads 1 fragment beyond it)
    const int64_t fixed = kFixedLds + 16, sums = kFixedLds + (int64_t)tl.tiles * 1024;
    const int64_t per_row = (int64_t)md->RS * 16;

    // Rows per workgroup and wavefronts: the least matrix and conversion work per
    // configuration (rows past the last of a group of 4, rows held twice) with two or more
    // workgroups on a CU.  A step costs its instructions' 16 cycles each and about 24
    // others' 4; a conversion about 160.
    const int Ly = g.L[1];
    const int64_t want = std::max<int64_t>(1, 512 / K);   // few configurations are spread over the chip
    const int most = (int)std::max<int64_t>(1, (Ly + want - 1) / want);
    double best = 0;
    int last_n = 0;
    const int fit = (int)std::min<int64_t>(most, (lds_budget / 2 - fixed) / per_row);   // (two workgroups on a CU)
    for (int ys0 = fit; ys0 >= 1; --ys0) {
        const int n = (Ly + ys0 - 1) / ys0;
        if (n == last_n) continue;
        last_n = n;
        int ys = (Ly + n - 1) / n;
        if (n > 1 && ys < most) ys = std::min(most, (ys + 3) / 4 * 4);   // whole quads
        const int chunks = (Ly + ys - 1) / ys;
        const int R = chunks == 1 ? Ly : ys + 1;
        const int64_t lds = std::max(fixed + per_row * R, sums);
        if (2 * lds > lds_budget) continue;
        const int items = (ys + 3) / 4 * md->W;
        const int64_t tasks = (int64_t)R * md->W * md->xs;
        for (int w = 4; w <= 8; w += 4) {   // (workgroups of 5 wavefronts leave SIMDs unused: 1.6 on a CU, not 3)
            const int on_cu = (int)std::min<int64_t>(lds_budget / lds, 16 / w);
            const double cost = (double)w * ((double)((items * md->xs + w - 1) / w) * (16.0 * tl.tiles + 96) +
                                             (double)((tasks + 64 * w - 1) / (64 * w)) * 640 + 1200);
            // fewer wavefronts on a CU hide less
            const double all = cost * chunks * (1.0 + 4.0 / (on_cu * w));
            if (best == 0 || all < best) {
                best = all;
                md->ys = ys;
                md->nchunks = chunks;
                md->R = R;
                md->threads = 64 * w;
                md->lds_bytes = (int)lds;
            }
        }
        if (best > 0 && n > 16 && want == 1) break;
    }
    if (best == 0) return false;
    // Shares of whole rows start a row once (about a third of a step); equal ones leave no
    // wavefront waiting: FCC 24^3 (18 items on 8 wavefronts) 142 -> 124 us, but FCC 20^3 (15
    // on 4) 561 -> 577 us.
    const int w = md->threads / 64, items = (md->ys + 3) / 4 * md->W;
    md->whole = (items + w - 1) / w * w * 8 <= items * 9;
    md->inv_xs = 1.0 / md->xs;
    md->inv_R = 1.0 / md->R;
    md->even = g.L[0] % 4 == 0 && Ly % 4 == 0 && md->ys % 4 == 0;
    // configurations per launch: their sums share the scratch
    md->step = (int32_t)mfma_configs_per_launch(md->threads, md->nchunks);
    if (md->nchunks > 1) {
        const int64_t bytes = K > (1 << 20) ? int64_t(1) << 20 : int64_t(8) << 20;
        md->step = (int32_t)std::max<int64_t>(8, bytes / (md->nchunks * kMfmaPartial * 4) / 8 * 8);
    }
    return (int64_t)md->ys * g.L[0] * g.L[2] <= kMfmaMaxCells;
}

size_t mfma_partial_bytes(const MfmaDesc &md, int64_t K) {
    return md.nchunks > 1 ? (size_t)std::min<int64_t>(K, md.step) * md.nchunks * kMfmaPartial * 4 : 0;
}

hipError_t launch_count_mfma(const MfmaDesc &md, int64_t K, const int8_t *species, int32_t *partial, int32_t *counts,
                             int32_t *bad, const double *tw, double *S_F, hipStream_t stream) {
    using KernelFn = void (*)(MfmaDesc, int64_t, const int8_t *, int32_t *, int32_t *, int32_t *, const double *,
                              double *);
    const bool q = md.even != 0;
    const KernelFn fn14 = q ? count_mfma_kernel<14, true> : count_mfma_kernel<14, false>;
    const KernelFn fn10 = q ? count_mfma_kernel<10, true> : count_mfma_kernel<10, false>;
    const KernelFn fn6 = q ? count_mfma_kernel<6, true> : count_mfma_kernel<6, false>;
    const KernelFn fn = md.tiles == 14 ? fn14 : md.tiles == 10 ? fn10 : fn6;
    hipError_t e = set_max_lds((const void *)fn, md.lds_bytes);
    if (e != hipSuccess) return e;
    const int E = md.S * md.M * md.M;
    const int64_t step = md.step;
    for (int64_t k0 = 0; k0 < K; k0 += step) {
        const int64_t kn = std::min(step, K - k0);
        const int64_t blocks = md.nchunks == 1 ? kn : (kn + 7) / 8 * 8 * md.nchunks;
        hipLaunchKernelGGL(fn, dim3((unsigned)blocks), dim3(md.threads), md.lds_bytes, stream, md, kn,
                           species + k0 * (int64_t)md.N, partial,
                           counts + k0 * (int64_t)E, bad + k0, tw, S_F ? S_F + 2 * k0 : nullptr);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        if (md.nchunks > 1) {
            hipLaunchKernelGGL(finalize_mfma_kernel, dim3((unsigned)kn),
                               dim3(md.nchunks > kFinalFew ? kFinalThreads : kFinishThreads), 0, stream, md,
                               partial, counts + k0 * (int64_t)E, bad + k0, tw,
                               S_F ? S_F + 2 * k0 : nullptr);
            if ((e = hipGetLastError()) != hipSuccess) return e;
        }
    }
    return hipSuccess;
}

}  // namespace pyhea
