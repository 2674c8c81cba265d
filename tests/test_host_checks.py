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


@pytest.mark.parametrize("lattice,L,M,S", [(0, (3, 3, 3), 4, 1), (0, (1, 2, 3), 4, 1), (0, (12, 12, 12), 5, 3),
                                           (0, (20, 20, 20), 5, 3), (1, (3, 3, 3), 4, 1), (1, (16, 16, 16), 5, 3),
                                           (0, (40, 40, 40), 4, 2)])
@pytest.mark.parametrize("K", [8, 2**20, 2**24 + 8, 2**27])
def test_one_launch_is_less_than_2_32_threads(lattice, L, M, S, K):
    out = np.zeros(5, np.int64)
    assert host_checks.lib().mfma_shape(lattice, _p(np.array(L, np.int32)), M, S, ctypes.c_int64(K), _p(out))
    threads, nchunks, step = (int(v) for v in out[:3])
    assert step >= 8 and step % 8 == 0
    assert step * nchunks * threads < 2**32


def test_the_evaluation_tests_run_on_the_matrix_cores():
    """What test_gpu_mfma_eval.py evaluates is counted by the kernel that it is about."""
    import test_gpu_mfma_eval as t

    def taken(lattice, L, M, S, K):
        out = np.zeros(5, np.int64)
        ok = host_checks.lib().mfma_shape(lattice, _p(np.array(L, np.int32)), M, S, ctypes.c_int64(K), _p(out))
        # (large cells with one row per workgroup, or in many workgroups, go to the bit-sliced
        # kernel if that covers them)
        return ok and (out[3] > 1 and out[1] <= 128 or np.prod(L) * (4, 2)[lattice] <= 1200000 or not out[4])

    assert all(taken(*c) for c in t.CASES)
    assert all(taken(*c, 1) for c in t.LARGE)
