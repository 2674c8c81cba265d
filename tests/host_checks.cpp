// Host side of the library, called by test_host_checks.py: the arithmetic and the launch
// shapes that kernels share with the host.
#include "geometry.h"
#include "sites.h"
#include "sro_bits.h"
#include "sro_mfma.h"

using namespace pyhea;

// Feature sums of pair sums H [4][4] (species 0-3), and back by the two passes that the
// sums of a whole configuration take.
extern "C" void feature_round_trip(const int64_t *H, int64_t *out) {
    const int64_t f[4][4] = {{1, 0, 0, 0}, {0, 2, 0, 2}, {0, 0, 4, 4}, {0, 2, 4, 8}};   // [feature][species], doubled
    MfmaSum F[16], G[16];
    for (int u = 0; u < 4; ++u)
        for (int v = 0; v < 4; ++v) {
            int64_t s = 0;
            for (int i = 0; i < 4; ++i)
                for (int j = 0; j < 4; ++j) s += f[u][i] * f[v][j] * H[4 * i + j];
            F[4 * u + v] = (MfmaSum)s;
        }
    for (int v = 0; v < 4; ++v) {
        MfmaSum a[4];
        species_of_features(F[v], F[4 + v], F[8 + v], F[12 + v], a);
        for (int i = 0; i < 4; ++i) G[4 * i + v] = a[i];
    }
    for (int i = 0; i < 4; ++i) {
        MfmaSum a[4];
        species_of_features(G[4 * i], G[4 * i + 1], G[4 * i + 2], G[4 * i + 3], a);
        for (int j = 0; j < 4; ++j) out[4 * i + j] = a[j];
    }
}

extern "C" void wrap_sites(const int32_t *r, int64_t n, int32_t m, int32_t *out) {
    for (int64_t i = 0; i < n; ++i) out[i] = wrap_site(r[i], m);
}

// The matrix-core kernel's launch shape for K configurations (160 KB of LDS): {threads,
// workgroups per configuration, configurations per launch, rows per workgroup, whether the
// bit-sliced kernel covers the cell too}; false if it is not taken.
extern "C" int mfma_shape(int lattice, const int *L, int M, int S, int64_t K, int64_t *out) {
    pyhea_lattice lat{};
    lat.lattice = lattice;
    for (int a = 0; a < 3; ++a) lat.L[a] = L[a];
    lat.n_species = M;
    lat.n_shells = S;
    Geometry g;
    std::string err;
    MfmaDesc md;
    if (build_geometry(&lat, &g, &err) != PYHEA_OK || !fill_mfma_desc(g, 160 * 1024, K, &md)) return 0;
    out[0] = md.threads;
    out[1] = md.nchunks;
    out[2] = md.step;
    out[3] = md.ys;
    BitDesc bd;
    out[4] = fill_bit_desc(g, 160 * 1024, K, 2, &bd);
    return 1;
}
