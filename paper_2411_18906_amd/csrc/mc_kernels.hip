// Persistent Monte Carlo kernel: SRO-targeted swap search (Sec. 4.2,
// Algorithm 3; Sec. 4.5-4.6).
//
// One workgroup runs one chain for up to `max_steps` steps.  Its configuration
// lies in a halo-padded copy in which a site's index is linear in its half-unit
// coordinates, so an offset is one delta for every site (geometry.h); a byte
// holds 5 times the species, the shift of the species' field in a neighbour
// histogram.
//
// A step:
//  1. Draw.  Candidates depend on counters only (Philox4x32-10, counter (slot,
//     step, chain, 0)), so the site pairs of kRing steps are drawn ahead by all
//     wavefronts side by side.
//  2. Evaluate.  A wavefront takes 32 candidates of one step and one shell, two
//     lanes per candidate: one lane per site gathers the species of its z_k
//     shell-k neighbours (all loads of up to 12 offsets in flight), and the two
//     lanes exchange histograms and evaluate one row of Eq. 4-5 each.
//  3. Rank.  Every wavefront forms dS = sum_k w_k dQ_k of all slots and ranks a
//     share of the improving ones by (dS, slot) (Eq. 6), then finds the earlier
//     candidates that a share of the ranks conflicts with.
//  4. Commit.  A conflict-free chunk of up to CH candidates in rank order is
//     re-validated as if every member commits: a half wavefront holds one (shell,
//     row) of the changed entries, a lane one member, prefix sums along the lanes
//     give the counts before each member, and each lane sums its row's term
//     changes in order.  Members before the first that fails commit -- exactly
//     what happens one by one, because a non-conflicting candidate's neighbour
//     histograms are unchanged -- and the walk goes on after the failed one.
//     BEST is a chunk of one member.
// After a step without a commit the wavefronts scan the following steps, a slot
// group each (a lane per candidate, all shells), until one holds an improving
// candidate; a chain that stays quiet hands its steps to the scan kernel.
// Counts are exact int32; every binary64 value is produced by the same
// expression sequence as the host contract, with contraction disabled.
//
// Bound: latency, one step after the other on one CU.  Every instruction that all
// wavefronts run costs their number in issue cycles, so 8 wavefronts measured
// better than 16 or 4 (FCC 20^3, 32 chains, 5 species, 3 shells: 35.4 ms of
// global search against 43.6 and 45.3), and constants sit in LDS or scalar
// registers because a descriptor load waits for L2.  FCC 40^3, 4 species, 2
// shells (1,450 committing steps, 19.6 commits each): 14.0 us per step with one
// wavefront per shell and 64 slots, commit walk in chunks of 16 and per-basis
// offset tables, 6.9 us now; of it evaluation 27 %, commits 39 %, ranks and
// conflicts 29 % (clocks of the first wavefront, its waits included).  512 chains of
// 250-16,000 sites: 6.1 -> 3.6 ms per call.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "device_common.h"
#include "mc_kernels.h"

namespace pyhea {

namespace {

template <bool kWide>
struct HistT {
    using type = uint32_t;
};
template <>
struct HistT<true> {
    using type = uint64_t;
};

// 5-bit fields: z_k <= 24 neighbours of one species per shell; a species' code
// is its field's shift
template <typename H>
__device__ __forceinline__ int fld(H h, int j) {
    return (int)((h >> (5 * j)) & 31u);
}
template <typename H>
__device__ __forceinline__ int fld_at(H h, int code) {
    return (int)((h >> code) & 31u);
}
// species of a code (codes 0, 5, .., 35)
__device__ __forceinline__ int species_of(int code) { return (code * 13) >> 6; }

__device__ __forceinline__ double sq_dev(int32_t n, double R, double t) {
    const double alpha = 1.0 - (double)n * R;
    const double d = alpha - t;
    return d * d;
}

// One (k, i, j) entry: the ratio R = N/(n_i n_j z_k), the target, the cached
// squared deviation and the exact pair count, read together (two 16-byte loads).
struct Ent {
    double R;
    double t;
    double sq;
    int32_t cnt;
    int32_t pad;
};

template <typename T>
__device__ __forceinline__ T pinned(T x) {
    static_assert(sizeof(T) == 4 || sizeof(T) == 8, "one or two dwords");
    uint32_t w[sizeof(T) / 4];
    __builtin_memcpy(w, &x, sizeof(T));
#pragma unroll
    for (size_t i = 0; i < sizeof(T) / 4; ++i) {
        w[i] = __builtin_amdgcn_readfirstlane(w[i]);
        asm volatile("" : "+s"(w[i]));
    }
    __builtin_memcpy(&x, w, sizeof(T));
    return x;
}

// A chain's constants, taken from its descriptor once: a load of the descriptor
// inside the step loop would wait for L2 every time.  What decides branches and
// loop bounds is held in scalar registers, the rest in LDS, where a broadcast
// read costs no register in between (scalar registers spilled in the chain
// kernel would be moved in and out of vector lanes).
struct Consts {
    double inv_Lx, inv_Ly;
    double w[kMaxShells];
    double tau;
    int64_t log_cap;
    uint32_t *log;
    int32_t lgA, Lx, Ly, Lz, hh, A2, B2, c0;
    int32_t P2[3];
    uint32_t N, key0, key1, chain_id;
    int32_t dl[kMaxOffsets], off_mod[kMaxOffsets];
};

struct Chain {
    int A, small_cell, sym;
    uint64_t zstart8;   // first offset of shell k in byte k (and the end of the last)
    uint32_t r2_8;      // squared radius of shell k in byte k
    const Consts *c;    // LDS, filled by the constructor; a barrier before the first use
    __device__ __forceinline__ Chain(const ChainDesc &d, Consts *lds)
        : A(pinned(d.A)), small_cell(pinned(d.small_cell)), sym(pinned(d.sym)), c(lds) {
        uint64_t z = 0;
        uint32_t r = 0;
#pragma unroll
        for (int k = 0; k <= kMaxShells; ++k) z |= (uint64_t)(uint32_t)d.zstart[k] << (8 * k);
#pragma unroll
        for (int k = 0; k < kMaxShells; ++k) r |= (uint32_t)(d.r2[k] & 0xFF) << (8 * k);
        zstart8 = pinned(z);
        r2_8 = pinned(r);
        for (int t = threadIdx.x; t < kMaxOffsets; t += blockDim.x) {
            lds->dl[t] = d.dl[t];
            lds->off_mod[t] = d.off_mod[t];
        }
        if (threadIdx.x == 0) {
            lds->inv_Lx = d.inv_Lx;
            lds->inv_Ly = d.inv_Ly;
            for (int k = 0; k < kMaxShells; ++k) lds->w[k] = d.w[k];
            lds->tau = d.tau;
            lds->log_cap = d.log_cap;
            lds->log = d.log;
            lds->lgA = d.lgA;
            lds->Lx = d.Lx;
            lds->Ly = d.Ly;
            lds->Lz = d.Lz;
            lds->hh = d.hh;
            lds->A2 = d.A2;
            lds->B2 = d.B2;
            lds->c0 = d.hh * (d.A2 + d.B2 + 1);
            for (int a = 0; a < 3; ++a) lds->P2[a] = d.P2[a];
            lds->N = d.N;
            lds->key0 = (uint32_t)d.seed;
            lds->key1 = (uint32_t)(d.seed >> 32);
            lds->chain_id = d.chain_id;
        }
    }
    __device__ __forceinline__ int zstart(int k) const { return (int)(zstart8 >> (8 * k)) & 0xFF; }
    __device__ __forceinline__ int r2(int k) const { return (int)(r2_8 >> (8 * k)) & 0xFF; }
};

constexpr int kMaxWindow = 64;   // steps the workgroup scans between two barriers at most

// LDS of a chain: a part of fixed layout, then arrays that follow B and CH (Ring).
template <int M>
struct alignas(16) Lds {
    Ent ent[kMaxShells * M * M];
    Consts c;
    uint64_t cm[kWave];      // earlier ranks each rank conflicts with
    double rowsum[kMaxShells * M * kChunk];   // change of a row's sum under each member of a chunk
    int32_t nulls;           // null draws of a window scanned by the whole chip
    int32_t found;           // a window's first step with an improving candidate
    uint8_t win_nulls[kMaxWindow * kMaxB / kWave];   // null draws per slot group of a window
};
struct Ring {
    uint2 *pos;         // [kRing][B] packed positions of p and q (10 bits per axis) of the steps drawn ahead
    uint32_t *ab;       // [B] code of p | code of q << 8 | null << 16 | drawn << 17
    void *h;            // [S][2][B] neighbour histograms of p and q, partner removed
    double *dQ;         // [S][B]
    int32_t *order;     // [B] slots by rank, then [B] committed slots of the step
    int32_t *prefix;    // [E][CH] change of an entry's count up to and with each member
    uint8_t *store;     // species store
};

__device__ __forceinline__ uint8_t *carve(uint8_t *&p, size_t bytes) {
    uint8_t *r = p;
    p += (bytes + 15) & ~size_t(15);
    return r;
}

// the species code (5 x species) at an index of the padded copy
template <int kStore>
__device__ __forceinline__ int load_code(const uint8_t *store, const int8_t *pad, int32_t pid) {
    if constexpr (kStore == kStoreLds8) {
        return store[pid];
    } else if constexpr (kStore == kStoreLds4) {
        const uint32_t w = reinterpret_cast<const uint32_t *>(store)[pid >> 3];
        const int s = (int)((w >> ((pid & 7) << 2)) & 0xFu);
        return s + (s << 2);
    } else {
        return (int)(uint8_t)pad[(uint32_t)pid];
    }
}

template <int kStore>
__device__ __forceinline__ void store_code(uint8_t *store, int8_t *pad, int32_t pid, int code) {
    if constexpr (kStore == kStoreLds8) {
        store[pid] = (uint8_t)code;
    } else if constexpr (kStore == kStoreLds4) {
        uint32_t *w = reinterpret_cast<uint32_t *>(store) + (pid >> 3);
        const int sh = (pid & 7) << 2;
        atomicAnd(w, ~(0xFu << sh));
        atomicOr(w, (uint32_t)species_of(code) << sh);
    } else {
        pad[(uint32_t)pid] = (int8_t)code;
    }
}

__device__ __forceinline__ uint32_t pack_pos(int x, int y, int z) {
    return (uint32_t)x | ((uint32_t)y << 10) | ((uint32_t)z << 20);
}

// packed half-unit position of a site id
__device__ __forceinline__ uint32_t pos_of_site(int A, const Consts &c, uint32_t p) {
    const SiteCoord s = site_coord(p, c.lgA, c.Lx, c.Ly, c.inv_Lx, c.inv_Ly);
    int bx, by, bz;
    basis_bits(A, s.b, bx, by, bz);
    return pack_pos(2 * s.cx + bx, 2 * s.cy + by, 2 * s.cz + bz);
}

// index of a packed position in the padded copy
__device__ __forceinline__ int32_t pid_of(const Consts &c, uint32_t pos) {
    return (int32_t)(__umul24((uint32_t)c.A2, pos >> 20) + __umul24((uint32_t)c.B2, (pos >> 10) & 1023u) +
                     (pos & 1023u) + (uint32_t)c.c0) >> 1;
}

// site id p = ((cz Ly + cy) Lx + cx) A + b of a packed position
__device__ __forceinline__ uint32_t site_id(int A, const Consts &c, uint32_t pos) {
    const int x = (int)(pos & 1023u), y = (int)((pos >> 10) & 1023u), z = (int)(pos >> 20);
    const int bx = x & 1, by = y & 1, bz = z & 1;
    // FCC basis (0,0,0), (1,1,0), (1,0,1), (0,1,1); BCC (0,0,0), (1,1,1)
    const int b = A == 2 ? bx : ((bx & by) ? 1 : ((bx & bz) ? 2 : ((by & bz) ? 3 : 0)));
    return (uint32_t)((((z >> 1) * c.Ly + (y >> 1)) * c.Lx + (x >> 1)) * A + b);
}

// squared minimum-image distance (half units) between two packed positions
__device__ __forceinline__ int min_image_r2(const Consts &c, uint32_t u, uint32_t v) {
    const int Ls[3] = {c.Lx, c.Ly, c.Lz};
    uint32_t r2 = 0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const int x = (int)((u >> (10 * a)) & 1023u) - (int)((v >> (10 * a)) & 1023u);
        const int y = x < 0 ? -x : x;
        const uint32_t m = (uint32_t)min(y, 2 * Ls[a] - y);
        r2 += __umul24(m, m);
    }
    return (int)r2;
}

// the packed (pos_q - pos_p) mod box, for the exact multiplicity count on small cells
__device__ __forceinline__ int32_t mod_delta(const Consts &c, uint32_t pp, uint32_t pq) {
    const int Ls[3] = {c.Lx, c.Ly, c.Lz};
    int32_t out = 0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        int x = (int)((pq >> (10 * a)) & 1023u) - (int)((pp >> (10 * a)) & 1023u);
        if (x < 0) x += 2 * Ls[a];
        out |= x << (10 * a);
    }
    return out;
}

// number of offsets t0 .. t1 - 1 (a shell's, r2 its squared radius) from p to q
__device__ __forceinline__ int partner_count(const Chain &d, uint32_t pp, uint32_t pq, int r2, int t0, int t1) {
    if (!d.small_cell) return min_image_r2(*d.c, pp, pq) == r2 ? 1 : 0;
    const int32_t md = mod_delta(*d.c, pp, pq);
    int m = 0;
    for (int t = t0; t < t1; ++t) m += d.c->off_mod[t] == md ? 1 : 0;
    return m;
}

// Does one of the sites up, uq lie on, or in shells 1..S of, one of vp, vq?  The
// shells are the S shortest lattice vector lengths, so a distance is one of them
// (or 0) exactly when it is no longer than the last; r2 = that length squared.
__device__ __forceinline__ bool conflict(const Consts &c, uint32_t up, uint32_t uq, uint32_t vp, uint32_t vq, int r2) {
    return min(min(min_image_r2(c, up, vp), min_image_r2(c, up, vq)),
               min(min_image_r2(c, uq, vp), min_image_r2(c, uq, vq))) <= r2;
}

// f(index in the padded copy) for a packed position and each of its halo copies
template <class F>
__device__ __forceinline__ void for_copies(const int Ls[3], const int P2[3], int hh, int A2, int B2, uint32_t pos, F f) {
    int c[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        c[a] = (int)((pos >> (10 * a)) & 1023u) + hh;
        while (c[a] >= Ls[a]) c[a] -= Ls[a];
    }
#pragma unroll 1
    for (int z = c[2]; z < P2[2]; z += Ls[2])
#pragma unroll 1
        for (int y = c[1]; y < P2[1]; y += Ls[1])
#pragma unroll 1
            for (int x = c[0]; x < P2[0]; x += Ls[0]) f((A2 * z + B2 * y + x) >> 1);
}

// species code v at a packed position and at every halo copy of it
template <int kStore>
__device__ __forceinline__ void write_site(uint8_t *store, int8_t *pad, const Consts &c, uint32_t pos, int v) {
    const int Ls[3] = {2 * c.Lx, 2 * c.Ly, 2 * c.Lz};
    const int P2[3] = {c.P2[0], c.P2[1], c.P2[2]};
    for_copies(Ls, P2, c.hh, c.A2, c.B2, pos, [&](int pid) { store_code<kStore>(store, pad, pid, v); });
}

// Histogram of the neighbours along offsets t0 .. t1 - 1 of the site at pid; all
// loads of a group of offsets are issued before the first is used.
template <int kStore, typename H>
__device__ __forceinline__ H gather(const uint8_t *store, const int8_t *pad, const Chain &d, int32_t pid, int t0,
                                    int t1) {
    H h = 0;
    auto group = [&](int t, auto n) {
        constexpr int kN = decltype(n)::value;
        int v[kN];
#pragma unroll
        for (int u = 0; u < kN; ++u) v[u] = load_code<kStore>(store, pad, pid + d.c->dl[t + u]);
#pragma unroll
        for (int u = 0; u < kN; ++u) h += (H)1 << v[u];
    };
    int t = t0;
#pragma unroll 1
    for (; t + 12 <= t1; t += 12) group(t, std::integral_constant<int, 12>{});
#pragma unroll 1
    for (; t + 6 <= t1; t += 6) group(t, std::integral_constant<int, 6>{});
#pragma unroll 1
    for (; t < t1; ++t) group(t, std::integral_constant<int, 1>{});
    return h;
}

// The lane beside this one in a pair of lanes (2 i, 2 i + 1).
__device__ __forceinline__ uint32_t pair_swap(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0xB1, 0xF, 0xF, true);   // quad_perm [1,0,3,2]
}
__device__ __forceinline__ uint64_t pair_swap(uint64_t x) {
    return ((uint64_t)pair_swap((uint32_t)(x >> 32)) << 32) | pair_swap((uint32_t)x);
}
__device__ __forceinline__ double pair_swap(double x) {
    return __longlong_as_double((long long)pair_swap((uint64_t)__double_as_longlong(x)));
}

// One row (species of code ci) of the change of a swap: own[j] = sq(N + dN) - sq(N)
// of entry (i, j) and their sum over j from +0.0.  The row belongs to one of the
// swapped species; co is the other one's code, X = u_i (c_q - c_p) with u_i = +1
// for the species at p and -1 for the one at q, so dN_ij = X_j, plus X_i at j = i
// and minus X_i at j = o.
template <int M, typename H>
__device__ __forceinline__ double swap_row(const Ent *row, H hx, H hy, int ci, int co, double *own) {
    const int Xi = fld_at(hx, ci) - fld_at(hy, ci);
    double sum = 0.0;
#pragma unroll
    for (int j = 0; j < M; ++j) {
        int dn = fld(hx, j) - fld(hy, j);
        dn += 5 * j == ci ? Xi : 0;
        dn -= 5 * j == co ? Xi : 0;
        const Ent e = row[j];
        own[j] = sq_dev(e.cnt + dn, e.R, e.t) - e.sq;
        sum = sum + own[j];
    }
    return sum;
}

// dQ_k = sum over rows i of (sum over j of sq(N + dN) - sq(N)) for swapping the
// species of codes ca (at p) and cb (at q), whose shell-k neighbour histograms
// (partner removed) are cp and cq; two lanes per candidate (side 0 and 1), both
// return the sum; ent are the shell's entries.
template <int M, typename H>
__device__ __forceinline__ double pair_dQ(const Ent *ent, H cp, H cq, int ca, int cb, int side, int sym) {
    double dQ = 0.0;
    if (sym) {
        // Symmetric N, dN, R and target: only the rows of the swapped species lo <
        // hi need evaluating (side 0 takes lo, side 1 hi); row i of the others
        // holds nonzero terms only at columns lo and hi, equal to entries (lo, i)
        // and (hi, i).  Terms with dN = 0 are exactly +0.0.
        const int lo = min(ca, cb), hi = max(ca, cb);
        const int ci = side ? hi : lo, co = side ? lo : hi;
        const bool at_p = ci == ca;
        double own[M];
        const double mine = swap_row<M, H>(ent + species_of(ci) * M, at_p ? cq : cp, at_p ? cp : cq, ci, co, own);
        const double other = pair_swap(mine);
        const double rlo = side ? other : mine, rhi = side ? mine : other;
#pragma unroll
        for (int i = 0; i < M; ++i) {
            const double both = own[i] + pair_swap(own[i]);
            dQ = dQ + (5 * i == lo ? rlo : (5 * i == hi ? rhi : both));
        }
    } else {
        // all rows, two at a time (side 0 the even ones)
        int D[M], u[M];
#pragma unroll
        for (int j = 0; j < M; ++j) {
            D[j] = fld(cq, j) - fld(cp, j);
            u[j] = (5 * j == ca ? 1 : 0) - (5 * j == cb ? 1 : 0);
        }
#pragma unroll
        for (int i0 = 0; i0 < M; i0 += 2) {
            const int i = min(i0 + side, M - 1);
            const int Di = i0 + 1 < M && side ? D[i0 + 1 < M ? i0 + 1 : i0] : D[i0];
            const int ui = i0 + 1 < M && side ? u[i0 + 1 < M ? i0 + 1 : i0] : u[i0];
            double rs = 0.0;
#pragma unroll
            for (int j = 0; j < M; ++j) {
                const Ent e = ent[i * M + j];
                const int dn = __mul24(ui, D[j]) + __mul24(u[j], Di);
                rs = rs + (sq_dev(e.cnt + dn, e.R, e.t) - e.sq);
            }
            const double other = pair_swap(rs);
            dQ = dQ + (side ? other : rs);
            if (i0 + 1 < M) dQ = dQ + (side ? rs : other);
        }
    }
    return dQ;
}

// inclusive prefix sum over each half wavefront
__device__ __forceinline__ int half_prefix_sum(int x) {
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xF, 0xF, true);   // row_shr:1
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xF, 0xF, true);   // row_shr:2
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xF, 0xF, true);   // row_shr:4
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xF, 0xF, true);   // row_shr:8
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xA, 0xF, false);  // row_bcast:15 into rows 1 and 3
    return x;
}

__device__ __forceinline__ uint64_t readlane_u64(uint64_t v, int l) {
    const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)v, l);
    const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(v >> 32), l);
    return ((uint64_t)hi << 32) | lo;
}

__device__ __forceinline__ void load_entries(Ent *ent, const ChainDesc &d, int E) {
    for (int e = threadIdx.x; e < E; e += blockDim.x) {
        Ent en;
        en.cnt = d.counts[e];
        en.R = d.R[e];
        en.t = d.target[e];
        en.sq = sq_dev(en.cnt, en.R, en.t);
        en.pad = 0;
        ent[e] = en;
    }
}

// A quiet chain's copy in HBM (its image), one code per byte whatever the store,
// from and to LDS: 16-byte blocks of an LDS byte store, eight codes per nibble
// word.
template <int kStore>
__device__ __forceinline__ void image_to_lds(uint8_t *store, const uint8_t *image, uint32_t Npad) {
    if constexpr (kStore == kStoreLds8) {
        for (uint32_t i = threadIdx.x; i < (Npad + 15) / 16; i += blockDim.x)
            reinterpret_cast<uint4 *>(store)[i] = reinterpret_cast<const uint4 *>(image)[i];
    } else {
        for (uint32_t i = threadIdx.x; i < (Npad + 7) / 8; i += blockDim.x) {
            const uint2 v = reinterpret_cast<const uint2 *>(image)[i];
            uint32_t w = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j)
                w |= (uint32_t)species_of((v.x >> (8 * j)) & 0xFF) << (4 * j) |
                     (uint32_t)species_of((v.y >> (8 * j)) & 0xFF) << (4 * j + 16);
            reinterpret_cast<uint32_t *>(store)[i] = w;
        }
    }
}
template <int kStore>
__device__ __forceinline__ void lds_to_image(uint8_t *image, const uint8_t *store, uint32_t Npad) {
    if constexpr (kStore == kStoreLds8) {
        for (uint32_t i = threadIdx.x; i < (Npad + 15) / 16; i += blockDim.x)
            reinterpret_cast<uint4 *>(image)[i] = reinterpret_cast<const uint4 *>(store)[i];
    } else {
        for (uint32_t i = threadIdx.x; i < (Npad + 7) / 8; i += blockDim.x) {
            const uint32_t w = reinterpret_cast<const uint32_t *>(store)[i];
            uint2 v = {0u, 0u};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                v.x |= 5u * ((w >> (4 * j)) & 0xFu) << (8 * j);
                v.y |= 5u * ((w >> (4 * j + 16)) & 0xFu) << (8 * j);
            }
            reinterpret_cast<uint2 *>(image)[i] = v;
        }
    }
}

// pair_dQ by one lane (the scan, where the whole chip is busy): the same terms and
// sums.
template <int M, typename H>
__device__ __forceinline__ double lane_dQ(const Ent *ent, H cp, H cq, int ca, int cb, int sym) {
    double dQ = 0.0;
    if (sym) {
        const int lo = min(ca, cb), hi = max(ca, cb);
        const bool lo_at_p = lo == ca;
        const H hx = lo_at_p ? cq : cp, hy = lo_at_p ? cp : cq;
        double dl[M], dh[M];
        const double rlo = swap_row<M, H>(ent + species_of(lo) * M, hx, hy, lo, hi, dl);
        const double rhi = swap_row<M, H>(ent + species_of(hi) * M, hy, hx, hi, lo, dh);
#pragma unroll
        for (int i = 0; i < M; ++i) dQ = dQ + (5 * i == lo ? rlo : (5 * i == hi ? rhi : dl[i] + dh[i]));
    } else {
        int D[M], u[M];
#pragma unroll
        for (int j = 0; j < M; ++j) {
            D[j] = fld(cq, j) - fld(cp, j);
            u[j] = (5 * j == ca ? 1 : 0) - (5 * j == cb ? 1 : 0);
        }
#pragma unroll
        for (int i = 0; i < M; ++i) {
            double rs = 0.0;
#pragma unroll
            for (int j = 0; j < M; ++j) {
                const Ent e = ent[i * M + j];
                const int dn = __mul24(u[i], D[j]) + __mul24(u[j], D[i]);
                rs = rs + (sq_dev(e.cnt + dn, e.R, e.t) - e.sq);
            }
            dQ = dQ + rs;
        }
    }
    return dQ;
}

// The candidates of one slot group (64 slots) of step `step`, a lane each with all
// its shells: *nulls the null draws among the first `tasks` slots; true if one
// improves.  dS is formed by the expressions of a chain's own evaluation in the
// same order.
template <int kStore, int M>
__device__ __forceinline__ bool scan_item(const Chain &d, const Ent *ent, const uint8_t *store, const int8_t *pad,
                                          int S, uint32_t step, int slot, int tasks, int *nulls) {
    using Hist = typename HistT<(M > 6)>::type;
    const Consts &c = *d.c;
    bool null_draw = false, imp = false;
    if (slot < tasks) {
        uint32_t x[4] = {(uint32_t)slot, step, c.chain_id, 0u};
        philox4x32_10(x, c.key0, c.key1);
        const uint32_t pp = pos_of_site(d.A, c, __umulhi(x[0], c.N)), pq = pos_of_site(d.A, c, __umulhi(x[1], c.N));
        const int32_t pidp = pid_of(c, pp), pidq = pid_of(c, pq);
        const int ca = load_code<kStore>(store, pad, pidp), cb = load_code<kStore>(store, pad, pidq);
        null_draw = ca == cb;
        if (!null_draw) {
            double dS = 0.0;
#pragma unroll 1
            for (int k = 0; k < S; ++k) {
                const int t0 = d.zstart(k), t1 = d.zstart(k + 1);
                Hist cp = gather<kStore, Hist>(store, pad, d, pidp, t0, t1);
                Hist cq = gather<kStore, Hist>(store, pad, d, pidq, t0, t1);
                const Hist m = (Hist)partner_count(d, pp, pq, d.r2(k), t0, t1);
                cp -= m << cb;
                cq -= m << ca;
                dS = dS + c.w[k] * lane_dQ<M, Hist>(ent + k * M * M, cp, cq, ca, cb, d.sym);
            }
            imp = dS < -c.tau;
        }
    }
    *nulls = (int)__popcll(ballot64(null_draw));
    return ballot64(imp) != 0;
}

constexpr int kMinScan = 48;    // steps left below which a quiet chain finishes by itself

// kGroups: slot groups of 64 (1, or kMaxB / 64 for any B); 0: one, with few candidates a
// step.  A window takes about as long as two to four steps by themselves, and with few
// candidates a chain often commits after that many steps; such a chain opens windows only
// after kFewGap quiet steps, or if as many came before its last commit.  ms for 64 chains of
// 2,000 steps, without / with that: FCC 20^3, 1 candidate 12.6 / 8.6, 4 candidates 15.2 / 11.9;
// BCC 10^3, 6 species, 4 shells 13.3 / 10.0; FCC 4^3, commits far apart, 2.06 / 2.05.
constexpr int kFewGap = 8;
template <int kStore, int M, int kGroups>
__global__ void __launch_bounds__(kMaxWaves * kWave, 4) mc_kernel(const ChainDesc *__restrict__ descs, int32_t max_steps, int32_t K,
                                                  int32_t CH, int32_t quiet) {
    using Hist = typename HistT<(M > 6)>::type;
    constexpr bool kFew = kGroups == 0;
    constexpr int kG = kFew ? 1 : kGroups;
    const ChainDesc &desc = descs[blockIdx.x];
    ChainState *st = desc.state;
    if (st->done) return;

    const int S = pinned(desc.S), E = S * M * M;
    const int B = pinned(desc.B);
    const int Gs = kG == 1 ? 1 : (B + kWave - 1) / kWave;   // slot groups of 64 and of 32
    const int Gh = (B + 31) / 32;
    const int nthreads = blockDim.x, nw = nthreads / kWave;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
    const int lane = threadIdx.x % kWave;
    const uint64_t below = (1ull << lane) - 1ull;
    uint64_t share = 0;   // slots l with l mod nw = wave
    for (int l = wave; l < kWave; l += nw) share |= 1ull << l;
    share = pinned(share);

    extern __shared__ __align__(16) uint8_t smem[];
    Lds<M> &L = *reinterpret_cast<Lds<M> *>(smem);
    Ring R;
    {
        uint8_t *p = smem + sizeof(Lds<M>);
        R.pos = (uint2 *)carve(p, kRing * B * 8);
        R.ab = (uint32_t *)carve(p, B * 4);
        R.h = carve(p, 2 * S * B * (int)sizeof(Hist));
        R.dQ = (double *)carve(p, S * B * 8);
        R.order = (int32_t *)carve(p, 2 * B * 4);
        R.prefix = (int32_t *)carve(p, E * CH * 4);
        R.store = p;
    }
    Hist *rec_h = (Hist *)R.h;   // [S][2][B]: of p, of q
    int32_t *list = R.order + B;
    const Chain d(desc, &L.c);
    const Consts &c = L.c;
    int8_t *pad = pinned(desc.pad_global);

    // ---- load chain state into LDS ------------------------------------------------
    load_entries(L.ent, desc, E);
    __syncthreads();
    const int scan_steps = st->scan_steps;   // > 0: back from a scanned window
    if (kStore != kStoreGlobal && scan_steps > 0) {
        image_to_lds<kStore>(R.store, desc.image, desc.Npad);
    } else if constexpr (kStore != kStoreGlobal) {
        if constexpr (kStore == kStoreLds4) {
            const int nword = (int)((desc.Npad + 7) / 8);
            for (int i = threadIdx.x; i < nword; i += nthreads) reinterpret_cast<uint32_t *>(R.store)[i] = 0;
            __syncthreads();
        }
        for (uint32_t p = threadIdx.x; p < desc.N; p += nthreads) {
            const int s = desc.species[p];
            const uint32_t pos = pos_of_site(d.A, c, p);
            if constexpr (kStore == kStoreLds4) {
                const int Ls[3] = {2 * c.Lx, 2 * c.Ly, 2 * c.Lz};
                const int P2[3] = {c.P2[0], c.P2[1], c.P2[2]};
                for_copies(Ls, P2, c.hh, c.A2, c.B2, pos, [&](int pid) {
                    atomicOr(reinterpret_cast<uint32_t *>(R.store) + (pid >> 3), (uint32_t)s << ((pid & 7) << 2));
                });
            } else {
                write_site<kStore>(R.store, pad, c, pos, 5 * s);
            }
        }
    }
    if (threadIdx.x == 0) L.nulls = 0;
    __syncthreads();

    // Chain counters, the same in every thread.  A step holds B trials but for the
    // chain's last, so trials follow from steps; left = steps to go.
    const int64_t n_trials = pinned(desc.n_trials);
    const int64_t n_steps = pinned((n_trials + B - 1) / B);
    const int last_tasks = pinned((int)(n_trials - (n_steps - 1) * B));
    int64_t commits = pinned(st->commits), step = pinned(st->steps), nulls = pinned(st->null_trials);
    int depth = __builtin_amdgcn_readfirstlane(st->depth);
    int stop_reason = 0;
    bool done = step >= n_steps;
    const int depth_limit = pinned(desc.depth_limit);
    const int r2max = d.r2(S - 1);
    const bool best = pinned(desc.mode) == PYHEA_MODE_BEST;
    const int chunk_max = best ? 1 : CH;
    const int scan_cap = quiet > 0 ? desc.scan_cap / Gs : 0;

    int steps_left = max_steps;
    // A step without a commit leaves the state as it was, so the steps after it are
    // independent until one commits: after such a step, with K > 1, the wavefronts
    // scan windows of `window` steps (0: none), one slot group each and no barrier
    // in between, up to the first step with an improving candidate.
    int window = 0;
    // A quiet chain hands its next steps to the scan kernel: with quiet > 0 it
    // leaves once `quiet` steps in a row committed nothing and at least
    // kMinScan are left, and comes back at the first step of the scanned window
    // that holds an improving candidate (or at its end).  The steps before it
    // commit nothing: only their counters move on.
    int quiet_run = 0, last_gap = 0;
    if (scan_steps > 0) {
        const int adv = __builtin_amdgcn_readfirstlane(st->scan_found);
        int32_t sum = 0;
        const int ng = adv * Gs;
        for (int i = threadIdx.x; i < ng; i += nthreads) sum += desc.scan_nulls[i];
#pragma unroll
        for (int m = 1; m < kWave; m <<= 1) sum += __shfl_xor(sum, m);
        if (lane == 0) atomicAdd(&L.nulls, sum);
        __syncthreads();
        nulls += __builtin_amdgcn_readfirstlane(L.nulls);
        step += adv;
        depth += adv;
        if (depth_limit > 0 && depth >= depth_limit) {
            stop_reason = PYHEA_STOP_DEPTH;
            done = true;
        } else if (step >= n_steps) {
            stop_reason = PYHEA_STOP_TRIALS;
            done = true;
        }
        if (adv == scan_steps) quiet_run = quiet;   // the window's end: scan on
    }
    int scan_next = 0;
    int64_t ring0 = step, ring_end = step;   // steps whose draws the ring holds
    while (!done && steps_left > 0) {
        if (quiet > 0 && quiet_run >= quiet) {
            int64_t left = n_steps - step;
            if (depth_limit > 0) left = min(left, (int64_t)(depth_limit - depth));
            if (left >= kMinScan) {
                scan_next = (int)min(left, (int64_t)scan_cap);
                break;
            }
        }
        if (window > 0) {
            int w = (int)min(n_steps - step, (int64_t)min(window, steps_left));
            if (depth_limit > 0) w = min(w, depth_limit - depth);
            if (threadIdx.x == 0) L.found = w;
            __syncthreads();
            for (int it = wave; it < w * Gs; it += nw) {
                const int rel = kG == 1 ? it : it / Gs;
                if (rel > __builtin_amdgcn_readfirstlane(L.found)) break;
                const int tasks = step + rel + 1 < n_steps ? B : last_tasks;
                int null_draws;
                const bool any = scan_item<kStore, M>(d, L.ent, R.store, pad, S, (uint32_t)step + (uint32_t)rel,
                                                      (it - rel * Gs) * kWave + lane, tasks, &null_draws);
                if (lane == 0) {
                    L.win_nulls[it] = (uint8_t)null_draws;
                    if (any) atomicMin(&L.found, rel);
                }
            }
            __syncthreads();
            const int adv = __builtin_amdgcn_readfirstlane(L.found);
            int sum = 0;
#pragma unroll
            for (int g = 0; g < kG; ++g)
                if (g * kWave + lane < adv * Gs) sum += L.win_nulls[g * kWave + lane];
#pragma unroll
            for (int m = 1; m < kWave; m <<= 1) sum += __shfl_xor(sum, m);
            nulls += __builtin_amdgcn_readfirstlane(sum);
            step += adv;
            depth += adv;
            quiet_run += adv;
            steps_left -= adv;
            if (depth_limit > 0 && depth >= depth_limit) {
                stop_reason = PYHEA_STOP_DEPTH;
                done = true;
            } else if (step >= n_steps) {
                stop_reason = PYHEA_STOP_TRIALS;
                done = true;
            }
            window = adv < w ? 0 : min(2 * window, kMaxWindow);
            __syncthreads();   // found and win_nulls are read until here
            continue;
        }
        const int tasks = step + 1 < n_steps ? B : last_tasks;

        // ---- 1. draw ahead ----------------------------------------------------------
        if (step >= ring_end) {
            ring0 = step;
            ring_end = step + kRing;
            for (int it = wave; it < kRing * Gs; it += nw) {
                const int kw = it / Gs, slot = (it - kw * Gs) * kWave + lane;
                if (slot < B) {
                    uint32_t x[4] = {(uint32_t)slot, (uint32_t)ring0 + (uint32_t)kw, c.chain_id, 0u};
                    philox4x32_10(x, c.key0, c.key1);
                    R.pos[kw * B + slot] = make_uint2(pos_of_site(d.A, c, __umulhi(x[0], c.N)),
                                                      pos_of_site(d.A, c, __umulhi(x[1], c.N)));
                }
            }
            __syncthreads();
        }
        const int ring_at = (int)(step - ring0) * B;   // the step's ring row

        // ---- 2. evaluate (32 slots, shell) ---------------------------------------------
        for (int it = wave; it < Gh * S; it += nw) {
            const int h = it / S, k = it - h * S;
            const int slot = h * 32 + (lane >> 1), side = lane & 1;
            const bool active = slot < tasks;
            uint32_t ab = 0;
            Hist own = 0;
            double dQ = 0.0;
            if (active) {
                const uint2 pos = R.pos[ring_at + slot];
                const uint32_t pp = pos.x, pq = pos.y;
                const int32_t pid = pid_of(c, side ? pq : pp);
                const int mine = load_code<kStore>(R.store, pad, pid);
                const int other = (int)pair_swap((uint32_t)mine);
                const int ca = side ? other : mine, cb = side ? mine : other;
                ab = (uint32_t)ca | ((uint32_t)cb << 8) | ((uint32_t)(ca == cb) << 16) | (1u << 17);
                if (ca != cb) {
                    const int t0 = d.zstart(k), t1 = d.zstart(k + 1);
                    own = gather<kStore, Hist>(R.store, pad, d, pid, t0, t1);
                    // without the partner: q is reached from p along m offsets of the shell
                    own -= (Hist)partner_count(d, pp, pq, d.r2(k), t0, t1) << other;
                    const Hist oth = pair_swap(own);
                    dQ = pair_dQ<M, Hist>(L.ent + k * M * M, side ? oth : own, side ? own : oth, ca, cb, side, d.sym);
                }
            }
            if (slot < B) {
                rec_h[(2 * k + side) * B + slot] = own;
                if (!side)
                    R.dQ[k * B + slot] = dQ;
                else if (k == 0)
                    R.ab[slot] = ab;
            }
        }
        __syncthreads();

        // ---- 3. rank ----------------------------------------------------------------------
        int n_impr = 0, step_nulls = 0;
        double dSg[kG];
        uint64_t mask[kG];
        const double tau = c.tau;
#pragma unroll
        for (int g = 0; g < kG; ++g) {
            mask[g] = 0;
            dSg[g] = 0.0;
            if (kG > 1 && g >= Gs) continue;
            const int s = g * kWave + lane;
            bool imp = false, nul = false;
            if (s < B) {
                const uint32_t ab = R.ab[s];
                double dS = 0.0;
#pragma unroll
                for (int q = 0; q < kMaxShells; ++q)
                    if (q < S) dS = dS + c.w[q] * R.dQ[q * B + s];
                dSg[g] = dS;
                nul = (ab >> 16) & 1u;   // null draws are drawn ones
                imp = ((ab >> 17) & 1u) && !nul && (dS < -tau);
            }
            mask[g] = ballot64(imp);
            step_nulls += (int)__popcll(ballot64(nul));
            n_impr += (int)__popcll(mask[g]);
        }
        int n_commit = 0;
        if (n_impr > 0) {

        // ranks: wavefront w takes the improving slots l with l mod nw = w
#pragma unroll
        for (int g = 0; g < kG; ++g) {
            if (kG > 1 && g >= Gs) continue;
            uint64_t m = mask[g] & share;
            while (m) {
                const int l = __ffsll((long long)m) - 1;
                m &= m - 1;
                const double du = readlane_f64(dSg[g], l);
                int rank = 0;
#pragma unroll
                for (int g2 = 0; g2 < kG; ++g2) {
                    if (kG > 1 && g2 >= Gs) continue;
                    const bool ahead = dSg[g2] < du || (dSg[g2] == du && (g2 < g || (g2 == g && lane < l)));
                    rank += (int)__popcll(ballot64(ahead) & mask[g2]);
                }
                if (lane == 0) R.order[rank] = g * kWave + l;
            }
        }
        __syncthreads();

        // ---- 4. commits, 64 ranks at a time -------------------------------------------
        for (int base = 0; base < n_impr; base += kWave) {
            const int nb = min(kWave, n_impr - base);
            const int my_s = lane < nb ? R.order[base + lane] : 0;
            const uint2 my_pos = R.pos[ring_at + my_s];
            const uint32_t my_p = my_pos.x, my_q = my_pos.y;
            bool out = lane >= nb;
            if (base > 0) {
                for (int n = 0; n < n_commit; ++n) {
                    const uint2 pos = R.pos[ring_at + list[n]];
                    out |= conflict(c, my_p, my_q, pos.x, pos.y, r2max);
                }
                __syncthreads();   // every wavefront has read cm
            }
            uint64_t my_cm = 0;
            if (!best && nb > 1) {
                for (int u = wave; u < nb; u += nw) {
                    const uint32_t up = __builtin_amdgcn_readlane(my_p, u), uq = __builtin_amdgcn_readlane(my_q, u);
                    const uint64_t mk = ballot64(lane < u && conflict(c, up, uq, my_p, my_q, r2max));
                    if (lane == 0) L.cm[u] = mk;
                }
                __syncthreads();
                if (lane < nb) my_cm = L.cm[lane];
            }
            const uint64_t valid = ballot64(!out);
            uint64_t committed = 0;
            int next = 0;
            for (;;) {
                // the greedy conflict-free set of the undecided ranks: those that
                // conflict with no committed and no undecided one, then the others
                // in rank order
                const uint64_t avail = next < kWave ? valid & (~0ull << next) : 0ull;
                const uint64_t blocked = ballot64(((avail >> lane) & 1ull) && (my_cm & (committed | avail)) != 0);
                uint64_t I = avail & ~blocked;
                for (uint64_t t = blocked; t; t &= t - 1) {
                    const int r = __ffsll((long long)t) - 1;
                    if ((readlane_u64(my_cm, r) & (committed | I)) == 0) I |= 1ull << r;
                }
                if (I == 0) break;
                // its first chunk_max members, member vi in lanes vi and vi + 32
                const bool in = (I >> lane) & 1ull;
                const int idx = (int)__popcll(I & below);
                const int m = min((int)__popcll(I), chunk_max);
                const int mem = __builtin_amdgcn_ds_permute((in && idx < m ? idx : kWave - 1) << 2, my_s);
                const int vi = lane & (kChunk - 1);
                const int slot = vi < m ? __builtin_amdgcn_ds_bpermute(vi << 2, mem) : 0;
                const uint32_t ab = R.ab[slot];
                const int ca = (int)(ab & 0xFFu), cb = (int)((ab >> 8) & 0xFFu);
                // each row's changes: a half wavefront per row, a lane per member
                for (int row0 = 2 * wave; row0 < S * M; row0 += 2 * nw) {
                    const int row = row0 + (lane >> 5);
                    const bool on = row < S * M && vi < m;
                    const int k = row / M, i = row - k * M;
                    Hist cp = 0, cq = 0;
                    if (on) {
                        cp = rec_h[2 * k * B + slot];
                        cq = rec_h[(2 * k + 1) * B + slot];
                    }
                    const int ui = (5 * i == ca ? 1 : 0) - (5 * i == cb ? 1 : 0);
                    const int Di = fld_at(cq, 5 * i) - fld_at(cp, 5 * i);
                    double sum = 0.0;
#pragma unroll
                    for (int j = 0; j < M; ++j) {
                        const int uj = (5 * j == ca ? 1 : 0) - (5 * j == cb ? 1 : 0);
                        int dn = __mul24(ui, fld(cq, j) - fld(cp, j)) + __mul24(uj, Di);
                        dn = on ? dn : 0;
                        const int incl = half_prefix_sum(dn);
                        if (on) {
                            const Ent en = L.ent[row * M + j];
                            const int after = en.cnt + incl;
                            double delta = 0.0;
                            if (dn != 0) delta = sq_dev(after, en.R, en.t) - sq_dev(after - dn, en.R, en.t);
                            sum = sum + delta;
                            R.prefix[(row * M + j) * CH + vi] = incl;
                        }
                    }
                    if (on) L.rowsum[row * kChunk + vi] = sum;
                }
                __syncthreads();
                // the first member whose dS fails (the step's first commit is not
                // re-validated); every wavefront finds the same one
                bool fails = false;
                if (lane < m) {
                    double dS = 0.0;
#pragma unroll
                    for (int k = 0; k < kMaxShells; ++k) {
                        if (k >= S) continue;
                        double Q = 0.0;
#pragma unroll
                        for (int i = 0; i < M; ++i) Q = Q + L.rowsum[(k * M + i) * kChunk + lane];
                        dS = dS + c.w[k] * Q;
                    }
                    fails = !(dS < -tau) && !(n_commit == 0 && lane == 0);
                }
                const uint64_t fm = ballot64(fails);
                const int f = fm ? __ffsll((long long)fm) - 1 : m;
                // members [0, f) commit: counts, squared deviations, sites and log
                if (f > 0)
                    for (int e = threadIdx.x; e < E; e += nthreads) {
                        const int dsum = R.prefix[e * CH + f - 1];
                        if (dsum != 0) {
                            Ent en = L.ent[e];
                            en.cnt += dsum;
                            en.sq = sq_dev(en.cnt, en.R, en.t);
                            L.ent[e] = en;
                        }
                    }
                if (wave == nw - 1 && vi < f) {
                    const bool second = lane >= kChunk;
                    const uint2 pos = R.pos[ring_at + slot];
                    write_site<kStore>(R.store, pad, c, second ? pos.y : pos.x, second ? ca : cb);
                }
                if (wave == 0 && lane < f) {
                    list[n_commit + lane] = slot;
                    const int64_t at = commits + n_commit + lane;
                    uint32_t *log = c.log;
                    if (log && at < c.log_cap) {
                        const uint2 pos = R.pos[ring_at + slot];
                        uint32_t *rec = log + 4 * at;
                        rec[0] = (uint32_t)step;
                        rec[1] = (uint32_t)slot;
                        rec[2] = site_id(d.A, c, pos.x);
                        rec[3] = site_id(d.A, c, pos.y);
                    }
                }
                n_commit += f;
                committed |= ballot64(in && idx < f);
                // on after the member that failed, or after the chunk
                next = __ffsll((long long)ballot64(in && idx == min(f, m - 1)));
                __syncthreads();
                if (best) break;
            }
            if (best) break;
        }
        commits += n_commit;

        }

        // ---- bookkeeping ------------------------------------------------------------------
        nulls += step_nulls;
        ++step;
        --steps_left;
        depth = n_commit > 0 ? 0 : depth + 1;
        if constexpr (kFew) last_gap = n_commit > 0 ? quiet_run : last_gap;
        quiet_run = n_commit > 0 ? 0 : quiet_run + 1;
        window = n_commit > 0 || K == 1 ? 0 : nw;
        if (kFew && max(last_gap, quiet_run) < kFewGap) window = 0;
        if (depth_limit > 0 && depth >= depth_limit) {
            stop_reason = PYHEA_STOP_DEPTH;
            done = true;
        } else if (step >= n_steps) {
            stop_reason = PYHEA_STOP_TRIALS;
            done = true;
        }
        if (n_impr == 0) __syncthreads();   // the records are read until here
    }

    // ---- write back -------------------------------------------------------------------
    for (int e = threadIdx.x; e < E; e += nthreads) desc.counts[e] = L.ent[e].cnt;
    if (kStore != kStoreGlobal && scan_next > 0) {
        lds_to_image<kStore>(desc.image, R.store, desc.Npad);
    } else if constexpr (kStore != kStoreGlobal) {
        for (uint32_t p = threadIdx.x; p < desc.N; p += nthreads)
            desc.species[p] = (int8_t)species_of(load_code<kStore>(R.store, pad, pid_of(c, pos_of_site(d.A, c, p))));
    }
    if (threadIdx.x == 0) {
        st->trials = min(step * B, n_trials);
        st->commits = commits;
        st->steps = step;
        st->null_trials = nulls;
        st->depth = depth;
        st->scan_steps = scan_next;
        st->scan_found = scan_next;
        if (done) {
            st->stop_reason = stop_reason;
            st->done = 1;
        }
    }
}

// The steps of a quiet chain's window, evaluated by the whole chip.  While
// nothing commits, the candidates of all later steps are evaluated against the
// same state (they are drawn from counters), so the steps of the window are
// independent: a wavefront takes one slot group (64 candidates of a step), a
// lane one candidate with all its shells, and no barrier is needed.  A group
// with an improving candidate lowers scan_found to its step; groups of later
// steps are skipped from then on, and every group of an earlier step is always
// evaluated, so that scan_found ends as the first such step and the null draws
// of all steps before it are complete.  dS is formed by the expressions of
// mc_kernel's phases 1 and 2 in the same order.
//
// Bound: VALU and LDS issue of the evaluation, spread over every CU instead of
// one.  FCC 20^3, 5 species, 3 shells, 10^6 trials (61 committing steps of
// 15,625, the last 30 of them far apart): 22.7 ms with every step on one CU, 1.9
// ms with windows; FCC 40^3, 10^7 trials: 244 -> 25 ms (both with the chain
// kernel of that time; 1.7-1.9 and 11-14 ms with today's).
template <int kStore, int M>
__global__ void __launch_bounds__(kScanThreads) scan_kernel(const ChainDesc *__restrict__ descs) {
    const ChainDesc &desc = descs[blockIdx.y];
    ChainState *st = desc.state;
    const int n_steps = st->scan_steps;
    if (st->done || n_steps == 0) return;
    const int S = desc.S, E = S * M * M, B = desc.B;
    const int Gs = (B + kWave - 1) / kWave;
    const int n_items = n_steps * Gs;
    constexpr int kWaves = kScanThreads / kWave;
    if ((int)blockIdx.x * kWaves >= n_items) return;
    const int lane = threadIdx.x % kWave;
    extern __shared__ __align__(16) uint8_t smem[];
    uint8_t *at = smem;
    Ent *ent = (Ent *)carve(at, E * sizeof(Ent));
    Consts *consts = (Consts *)carve(at, sizeof(Consts));
    uint8_t *store = at;
    // kStoreGlobal also scans chains that hold nibbles: their image is read in place
    const int8_t *pad = desc.store == kStoreGlobal ? desc.pad_global : (const int8_t *)desc.image;
    load_entries(ent, desc, E);
    const Chain d(desc, consts);

    if constexpr (kStore != kStoreGlobal) image_to_lds<kStore>(store, desc.image, desc.Npad);
    __syncthreads();

    const int64_t trials_left = desc.n_trials - pinned(st->trials);
    const int full = (int)min(trials_left / B, (int64_t)n_steps);   // steps of the window with B trials
    const int last_tasks = full < n_steps ? (int)(trials_left - (int64_t)full * B) : 0;
    const uint32_t step0 = (uint32_t)__builtin_amdgcn_readfirstlane((int32_t)st->steps);
    uint8_t *scan_nulls = desc.scan_nulls;
    const int stride = (int)gridDim.x * kWaves;
    int found = n_steps;   // read one item late: a stale value only costs work
#pragma unroll 1
    for (int it = (int)blockIdx.x * kWaves + __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave); it < n_items;
         it += stride) {
        const int rel = it / Gs;
        if (rel > found) break;
        const int seen = __hip_atomic_load(&st->scan_found, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        int nnull;
        const bool any = scan_item<kStore, M>(d, ent, store, pad, S, step0 + (uint32_t)rel,
                                              (it - rel * Gs) * kWave + lane, rel < full ? B : last_tasks, &nnull);
        if (lane == 0) {
            scan_nulls[it] = (uint8_t)nnull;
            if (any) atomicMin(&st->scan_found, rel);
        }
        found = any ? min(seen, rel) : seen;
    }
}

// Chain states of many chains into one contiguous array (one read-back).
__global__ void gather_states_kernel(const ChainDesc *__restrict__ descs, int n, ChainState *__restrict__ out) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = *descs[i].state;
}

__device__ __forceinline__ uint32_t desc_pos(const ChainDesc &d, uint32_t p) {
    const SiteCoord s = site_coord(p, d.lgA, d.Lx, d.Ly, d.inv_Lx, d.inv_Ly);
    int bx, by, bz;
    basis_bits(d.A, s.b, bx, by, bz);
    return pack_pos(2 * s.cx + bx, 2 * s.cy + by, 2 * s.cz + bz);
}

// padded HBM copy <-> unpadded configuration (HBM-resident chains)
__global__ void pad_fill_kernel(const ChainDesc *__restrict__ descs) {
    const ChainDesc &d = descs[blockIdx.y];
    if (d.store != kStoreGlobal || d.state->status != 0) return;
    const int Ls[3] = {2 * d.Lx, 2 * d.Ly, 2 * d.Lz};
    for (uint32_t p = blockIdx.x * blockDim.x + threadIdx.x; p < d.N; p += gridDim.x * blockDim.x) {
        const int v = 5 * d.species[p];
        for_copies(Ls, d.P2, d.hh, d.A2, d.B2, desc_pos(d, p), [&](int pid) { d.pad_global[pid] = (int8_t)v; });
    }
}

__global__ void pad_drain_kernel(const ChainDesc *__restrict__ descs) {
    const ChainDesc &d = descs[blockIdx.y];
    if (d.store != kStoreGlobal || d.state->status != 0) return;
    for (uint32_t p = blockIdx.x * blockDim.x + threadIdx.x; p < d.N; p += gridDim.x * blockDim.x) {
        const uint32_t pos = desc_pos(d, p);
        const int pid = (d.A2 * ((int)(pos >> 20) + d.hh) + d.B2 * ((int)((pos >> 10) & 1023u) + d.hh) +
                         (int)(pos & 1023u) + d.hh) >> 1;
        d.species[p] = (int8_t)species_of((uint8_t)d.pad_global[pid]);
    }
}

}  // namespace

template <int kStore, int kG>
const void *mc_fn(int M) {
    switch (M) {
        case 2: return (const void *)mc_kernel<kStore, 2, kG>;
        case 3: return (const void *)mc_kernel<kStore, 3, kG>;
        case 4: return (const void *)mc_kernel<kStore, 4, kG>;
        case 5: return (const void *)mc_kernel<kStore, 5, kG>;
        case 6: return (const void *)mc_kernel<kStore, 6, kG>;
        case 7: return (const void *)mc_kernel<kStore, 7, kG>;
        default: return (const void *)mc_kernel<kStore, 8, kG>;
    }
}
// From 16 candidates a step on windows from the first quiet step measured as well: FCC 20^3
// 11.6 ms without / 11.4 with the wait, BCC 10^3 5.9 / 5.6, FCC 4^3 1.57 / 1.58.
constexpr int kFewB = 16;
template <int kStore>
const void *mc_fn(int M, int B) {
    return B < kFewB ? mc_fn<kStore, 0>(M) : B <= kWave ? mc_fn<kStore, 1>(M) : mc_fn<kStore, kMaxB / kWave>(M);
}

int lds_fixed_bytes(int M) {
    switch (M) {
        case 2: return (int)sizeof(Lds<2>);
        case 3: return (int)sizeof(Lds<3>);
        case 4: return (int)sizeof(Lds<4>);
        case 5: return (int)sizeof(Lds<5>);
        case 6: return (int)sizeof(Lds<6>);
        case 7: return (int)sizeof(Lds<7>);
        default: return (int)sizeof(Lds<8>);
    }
}

int mc_lds_bytes(int S, int M, int B, int CH) {
    auto r = [](int b) { return (b + 15) & ~15; };
    const int E = S * M * M;
    int n = lds_fixed_bytes(M);
    n += r(kRing * B * 8);                       // pos
    n += r(B * 4);                               // ab
    n += r(2 * S * B * (M > 6 ? 8 : 4));         // h
    n += r(S * B * 8);                           // dQ
    n += r(2 * B * 4);                           // order, list
    n += r(E * CH * 4);                          // prefix
    return n;
}

int scan_lds_bytes(int S, int M) { return S * M * M * (int)sizeof(Ent) + (((int)sizeof(Consts) + 15) & ~15); }

hipError_t launch_mc(const ChainDesc *descs_dev, int n_chains, int store, int M, int B, int waves, int K, int CH,
                     int lds_bytes, int max_steps, hipStream_t stream, int quiet) {
    if (waves < 1 || waves > kMaxWaves || K < 1 || K > kMaxLookahead || CH < 1 || CH > kChunk)
        return hipErrorInvalidValue;
    const dim3 grid(n_chains), block(waves * kWave);
    const void *fn = store == kStoreLds8 ? mc_fn<kStoreLds8>(M, B)
                     : store == kStoreLds4 ? mc_fn<kStoreLds4>(M, B)
                                           : mc_fn<kStoreGlobal>(M, B);
    hipError_t e = set_max_lds(fn, lds_bytes);
    if (e != hipSuccess) return e;
    void *args[] = {(void *)&descs_dev, (void *)&max_steps, (void *)&K, (void *)&CH, (void *)&quiet};
    return hipLaunchKernel(fn, grid, block, args, (size_t)lds_bytes, stream);
}

template <int kStore>
const void *scan_fn(int M) {
    switch (M) {
        case 2: return (const void *)scan_kernel<kStore, 2>;
        case 3: return (const void *)scan_kernel<kStore, 3>;
        case 4: return (const void *)scan_kernel<kStore, 4>;
        case 5: return (const void *)scan_kernel<kStore, 5>;
        case 6: return (const void *)scan_kernel<kStore, 6>;
        case 7: return (const void *)scan_kernel<kStore, 7>;
        default: return (const void *)scan_kernel<kStore, 8>;
    }
}

hipError_t launch_scan(const ChainDesc *descs_dev, int n_chains, int store, int M, int store_bytes, int S,
                       int blocks_per_chain, hipStream_t stream) {
    if (n_chains < 1 || n_chains > 65535 || blocks_per_chain < 1) return hipErrorInvalidValue;
    // a configuration held as nibbles leaves no room for a second workgroup on its
    // CU; the scan reads it from HBM instead
    const bool in_lds = store == kStoreLds8;
    const void *fn = in_lds ? scan_fn<kStoreLds8>(M) : scan_fn<kStoreGlobal>(M);
    const size_t lds = (size_t)scan_lds_bytes(S, M) + (in_lds ? (size_t)store_bytes : 0);
    hipError_t e = set_max_lds(fn, lds);
    if (e != hipSuccess) return e;
    void *args[] = {(void *)&descs_dev};
    return hipLaunchKernel(fn, dim3(blocks_per_chain, n_chains), dim3(kScanThreads), args, lds, stream);
}

hipError_t launch_gather_states(const ChainDesc *descs_dev, int n_chains, ChainState *out, hipStream_t stream) {
    if (n_chains <= 0) return hipSuccess;
    hipLaunchKernelGGL(gather_states_kernel, dim3((n_chains + 255) / 256), dim3(256), 0, stream, descs_dev, n_chains,
                       out);
    return hipGetLastError();
}

// Species totals and the ratio table R = N / (n_i n_j z_k) of each chain from
// its initial pair counts (Eq. 2; n_i = row sum of shell 1 / z_1, one exact
// integer product and one IEEE division per entry).  A chain with an invalid id
// or an absent species is marked done with status EINVAL and left untouched.
__global__ void chain_ratio_kernel(const ChainDesc *__restrict__ descs, int n, const int32_t *__restrict__ bad) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const ChainDesc &d = descs[i];
    const int M = d.M, S = d.S;
    int64_t nsp[kMaxSpecies];
    bool ok = bad[i] == 0;
    for (int a = 0; a < M; ++a) {
        int64_t r = 0;
        for (int b = 0; b < M; ++b) r += d.counts[a * M + b];
        nsp[a] = r / d.zk[0];
        ok = ok && nsp[a] > 0;
    }
    if (!ok) {
        d.state->status = PYHEA_EINVAL;
        d.state->done = 1;
        return;
    }
    double *R = const_cast<double *>(d.R);
    for (int k = 0; k < S; ++k)
        for (int a = 0; a < M; ++a)
            for (int b = 0; b < M; ++b)
                R[(k * M + a) * M + b] = (double)d.N / (double)(nsp[a] * nsp[b] * (int64_t)d.zk[k]);
}

hipError_t launch_chain_ratio(const ChainDesc *descs_dev, int n_chains, const int32_t *bad, hipStream_t stream) {
    if (n_chains <= 0) return hipSuccess;
    hipLaunchKernelGGL(chain_ratio_kernel, dim3((n_chains + 63) / 64), dim3(64), 0, stream, descs_dev, n_chains, bad);
    return hipGetLastError();
}

hipError_t launch_pad_fill(const ChainDesc *descs_dev, int n_chains, hipStream_t stream) {
    hipLaunchKernelGGL(pad_fill_kernel, dim3(64, n_chains), dim3(256), 0, stream, descs_dev);
    return hipGetLastError();
}

hipError_t launch_pad_drain(const ChainDesc *descs_dev, int n_chains, hipStream_t stream) {
    hipLaunchKernelGGL(pad_drain_kernel, dim3(64, n_chains), dim3(256), 0, stream, descs_dev);
    return hipGetLastError();
}

}  // namespace pyhea
