"""Arithmetic that kernels share with the host, at the edges of its ranges (CPU)."""
import ctypes

import numpy as np
import pytest

import host_checks


def _p(a):
    return ctypes.c_void_p(a.ctypes.data)


@pytest.mark.parametrize("species", range(4))
@pytest.mark.parametrize("total", [1 << 26, (1 << 26) + 2, 1 << 27, (1 << 30) - 2])
def test_pair_sums_of_large_cells(species, total):
    """Half counts up to N z / 2 < 2^30, nearly all of one species: nothing wraps on the
    way from features to species."""
    H = np.arange(1, 17, dtype=np.int64).reshape(4, 4)
    H[species, species] = total - H.sum()
    H[(species + 1) % 4, species] = total // 7
    out = np.empty_like(H)
    host_checks.lib().feature_round_trip(_p(H), _p(out))
    np.testing.assert_array_equal(out, H)



@pytest.mark.parametrize("m", [2, 6, 20, 80, 1022])
def test_decoded_sites_stay_in_the_box(m):
    """Whatever a position decodes to is a coordinate of the box, its residue modulo m."""
    r = np.concatenate([np.arange(-3 * m - 3, 3 * m + 4), [-2**31, -2**31 + 1, 2**31 - 1, -4096, 4096, -128, 64],
                        np.random.default_rng(m).integers(-2**31, 2**31, 1000)]).astype(np.int32)
    out = np.empty_like(r)
    host_checks.lib().wrap_sites(_p(r), ctypes.c_int64(len(r)), m, _p(out))
    np.testing.assert_array_equal(out, r.astype(np.int64) % m)
