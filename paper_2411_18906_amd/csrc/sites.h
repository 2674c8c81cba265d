// Nearest-site assignment of external structures: descriptor and launcher.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pyhea {

struct SiteMapDesc {
    int32_t lattice;     // PYHEA_FCC or PYHEA_BCC
    int32_t A;           // sites per conventional cell
    int32_t L[3];
    int32_t M;           // species ids must lie in [0, M)
    int64_t N;           // sites
    double scale[3];     // half lattice units per unit of length, per axis (2 L / box)
    double w[3];         // squared length of a half unit, 1 / scale^2
    double max_disp2;    // squared largest accepted displacement (length units)
};

// r modulo m, in [0, m).  Positions reduced into the box decode to -1 .. m + 1, so the
// division is rare; but beyond about 2^53 periods the reduction in binary64 leaves any
// residual, and the site must still be one of the box's.
__host__ __device__ inline int wrap_site(int r, int m) {
    if ((unsigned)r < (unsigned)m) return r;
    r %= m;
    return r < 0 ? r + m : r;
}

// owner [N] int32 is device scratch (the entry point's or the caller's); flags [3]
// int32 is host memory, zero before the launch: {displacement too large, type out of
// range, vacant site}.  Writes species [N].
hipError_t launch_map_sites(const SiteMapDesc &md, int64_t n, const double *xyz, const int8_t *types,
                            int32_t *owner, int32_t *flags, int8_t *species, hipStream_t stream);

}  // namespace pyhea
