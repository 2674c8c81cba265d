"""The full evaluation on the matrix cores (the automatic choice for most of 4
and 5 species): counts, S and F equal to the oracle where the layout's remainders lie
-- rows of 1 to 9 columns (quarters of unequal length), 1 to 65 layers (words and
fragments half filled, wraps inside a word and between fragments), one row,
configurations cut into rows of workgroups, single ones spread over the chip, all
numbers of species and shells, any start address, invalid and absent species."""
import numpy as np
import pytest

from oracle import oracle as orc
from paper_2411_18906_amd import binding as pb
from paper_2411_18906_amd import workloads as wl

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

CASES = [
    # rows: quarters of 1 to 3 columns, some empty
    (orc.FCC, (1, 2, 3), 4, 1, 5), (orc.FCC, (2, 2, 2), 4, 2, 6), (orc.FCC, (3, 4, 5), 5, 3, 7),
    (orc.FCC, (4, 4, 4), 4, 2, 40), (orc.FCC, (5, 3, 4), 5, 4, 5), (orc.FCC, (9, 3, 2), 4, 3, 4),
    (orc.FCC, (8, 5, 3), 5, 3, 4), (orc.FCC, (13, 1, 6), 4, 1, 4),
    # layers: one to three fragments per column, last word and nibble anywhere
    (orc.FCC, (3, 3, 1), 5, 1, 4), (orc.FCC, (4, 3, 7), 4, 3, 4), (orc.FCC, (4, 3, 8), 5, 3, 4),
    (orc.FCC, (5, 3, 9), 5, 2, 4), (orc.FCC, (4, 3, 31), 5, 3, 4), (orc.FCC, (4, 3, 32), 5, 3, 4),
    (orc.FCC, (4, 3, 33), 5, 3, 4), (orc.FCC, (5, 4, 36), 4, 3, 4), (orc.FCC, (4, 3, 40), 4, 2, 4),
    (orc.FCC, (3, 3, 64), 5, 4, 4), (orc.FCC, (3, 3, 65), 5, 3, 4), (orc.FCC, (3, 3, 95), 5, 2, 4),
    # whole configurations per workgroup, and cut into rows
    (orc.FCC, (20, 20, 20), 5, 3, 600), (orc.FCC, (40, 40, 40), 4, 2, 600), (orc.FCC, (27, 41, 23), 5, 3, 520),
    (orc.FCC, (64, 64, 64), 5, 3, 3), (orc.FCC, (31, 33, 65), 2, 3, 3), (orc.FCC, (32, 32, 32), 3, 4, 4),
    (orc.FCC, (24, 24, 24), 5, 3, 600),
    # BCC, shells 1-3
    (orc.BCC, (31, 31, 31), 5, 3, 520), (orc.BCC, (32, 32, 32), 4, 2, 520), (orc.BCC, (1, 3, 3), 4, 1, 6),
    (orc.BCC, (2, 3, 3), 4, 3, 7), (orc.BCC, (9, 2, 7), 4, 3, 9), (orc.BCC, (5, 3, 2), 4, 3, 7),
    (orc.BCC, (3, 3, 1), 5, 1, 8), (orc.BCC, (6, 7, 37), 5, 3, 4), (orc.BCC, (48, 50, 66), 5, 3, 3),
    (orc.BCC, (8, 4, 64), 5, 2, 5),
]


@pytest.mark.parametrize("lattice,L,M,S,K", CASES)
def test_batch_equals_oracle(lattice, L, M, S, K):
    N = orc.n_sites(lattice, L)
    cfg = wl.iid_configs(N, M, min(K, 24), seed=K)
    reps = [np.roll(cfg, 4 * r, axis=1) for r in range(-(-K // len(cfg)))]
    cfg = np.concatenate(reps)[:K]
    cfg[1, :] = 0                      # species missing -> NaN
    cfg[2, 5] = M                      # ids out of range -> NaN
    if K > 3:
        cfg[3, N - 1] = -1
    rng = np.random.default_rng(1)
    tgt = rng.uniform(-0.2, 0.2, (S, M, M))
    w = rng.uniform(0.1, 1.0, S)
    counts = torch.zeros((K, S, M, M), dtype=torch.int32, device="cuda")
    SF = torch.zeros((K, 2), dtype=torch.float64, device="cuda")
    pb.pyhea_sro_eval_batch(lattice, L, M, S, torch.from_numpy(cfg).cuda(), counts, tgt, w, SF)
    torch.cuda.synchronize()
    c, sf = counts.cpu().numpy(), SF.cpu().numpy()
    which = list(range(min(K, 8))) + list(range(8, K, max(1, K // 6))) + [K - 1]
    for k in which:
        if k in (1, 2, 3) or (np.bincount(cfg[k], minlength=M) == 0).any():
            assert np.all(np.isnan(sf[k])), k
            continue
        want = orc.counts(lattice, L, M, S, cfg[k])
        np.testing.assert_array_equal(c[k], want, err_msg=str(k))
        _, _, S_o, F_o = orc.alpha_objective(lattice, L, M, S, cfg[k], want, tgt, w)
        assert sf[k, 0] == S_o and sf[k, 1] == F_o, k


@pytest.mark.parametrize("shift", [1, 2, 3])
@pytest.mark.parametrize("lattice,L", [(orc.FCC, (7, 3, 4)), (orc.BCC, (7, 3, 4))])
def test_any_start_address(lattice, L, shift):
    N, K, M, S = orc.n_sites(lattice, L), 5, 5, 3
    cfg = wl.iid_configs(N, M, K, seed=shift)
    buf = torch.zeros(K * N + 8, dtype=torch.int8, device="cuda")
    view = buf[shift:shift + K * N].view(K, N)
    view.copy_(torch.from_numpy(cfg).cuda())
    counts = torch.zeros((K, S, M, M), dtype=torch.int32, device="cuda")
    pb.pyhea_sro_eval_batch(lattice, L, M, S, view, counts)
    c = counts.cpu().numpy()
    for k in range(K):
        np.testing.assert_array_equal(c[k], orc.counts(lattice, L, M, S, cfg[k]))


@pytest.mark.parametrize("lattice,L,M,S", [(orc.FCC, (20, 20, 20), 5, 3), (orc.FCC, (40, 40, 40), 4, 2),
                                           (orc.BCC, (31, 31, 31), 5, 3), (orc.FCC, (64, 50, 70), 3, 4)])
def test_one_configuration(lattice, L, M, S):
    sp = wl.iid_configs(orc.n_sites(lattice, L), M, 1, seed=2)[0]
    t, w = np.zeros((S, M, M)), np.ones(S)
    counts, alpha, S_, F = pb.pyhea_sro_eval(lattice, L, M, S, torch.from_numpy(sp).cuda(), t, w)
    want = orc.counts(lattice, L, M, S, sp)
    np.testing.assert_array_equal(counts, want)
    a_o, _, S_o, F_o = orc.alpha_objective(lattice, L, M, S, sp, want, t, w)
    np.testing.assert_array_equal(alpha, a_o)
    assert S_ == S_o and F == F_o


@pytest.mark.parametrize("lattice,L,S,K", [(orc.FCC, (40, 40, 40), 3, 2), (orc.FCC, (20, 20, 20), 4, 600),
                                           (orc.BCC, (31, 31, 31), 3, 600)])
@pytest.mark.parametrize("most", [0, 3, 4])
def test_nearly_one_species(lattice, L, S, K, most):
    """The largest sums a feature product can reach (species 3) stay exact."""
    N = orc.n_sites(lattice, L)
    sp = np.full(N, most, np.int8)
    sp[np.random.default_rng(most).choice(N, 40, replace=False)] = np.arange(40) % 5
    counts = torch.zeros((K, S, 5, 5), dtype=torch.int32, device="cuda")
    pb.pyhea_sro_eval_batch(lattice, L, 5, S, torch.from_numpy(sp).cuda().repeat(K, 1), counts)
    want = orc.counts(lattice, L, 5, S, sp)
    c = counts.cpu().numpy()
    for k in (0, K - 1):
        np.testing.assert_array_equal(c[k], want)


def test_fixed_scratch_limit_is_the_same_for_every_kernel():
    """A batch is refused by the fixed scratch for the same numbers of configurations
    whichever kernel counts it."""
    lattice, L, M, S = orc.FCC, (40, 40, 40), 4, 2
    N = orc.n_sites(lattice, L)

    def refused(K, kernel):
        pb.pyhea_tune_force_eval(kernel)
        try:
            pb.pyhea_sro_eval_batch_noalloc(lattice, L, M, S, species[:K], counts[:K])
            torch.cuda.synchronize()
            return False
        except pb.PyheaError:
            return True
        finally:
            pb.pyhea_tune_force_eval(-1)

    most = 130000         # flags and two bit-sliced workgroups' 64 bytes each: 17.2 MB > the 16 MiB array
    species = torch.zeros((most, N), dtype=torch.int8, device="cuda")
    counts = torch.zeros((most, S, M, M), dtype=torch.int32, device="cuda")
    got = [(refused(K, -1), refused(K, 1)) for K in (100, 4096, most)]
    assert all(a == b for a, b in got) and not got[0][0] and not got[1][0] and got[2][0]


LARGE = [(orc.FCC, (200, 200, 20), 5, 3), (orc.FCC, (60, 511, 60), 5, 4), (orc.FCC, (128, 511, 32), 5, 3),
         (orc.FCC, (128, 511, 32), 4, 3)]


@pytest.mark.parametrize("lattice,L,M,S", LARGE)
@pytest.mark.parametrize("fractions", [(0.01, 0.01, 0.01, 0.96, 0.01), (0.05, 0.05, 0.05, 0.8, 0.05)])
def test_large_cells(lattice, L, M, S, fractions):
    """N z of 2^26 to 2^28: 64 quarter units a pair are more than 32 bits hold."""
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    p = torch.tensor(fractions[5 - M:], device="cuda")
    edges = torch.cumsum(p / p.sum(), 0)[:-1]
    u = torch.rand(orc.n_sites(lattice, L), device="cuda", generator=g)
    sp = torch.bucketize(u, edges).to(torch.int8).unsqueeze(0)
    got = torch.zeros((2, S, M, M), dtype=torch.int32, device="cuda")
    pb.pyhea_sro_eval_batch(lattice, L, M, S, sp, got[:1])
    pb.pyhea_tune_force_eval(0)
    try:
        pb.pyhea_sro_eval_batch(lattice, L, M, S, sp, got[1:])
    finally:
        pb.pyhea_tune_force_eval(-1)
    torch.cuda.synchronize()
    assert torch.equal(got[0], got[1])


@pytest.mark.parametrize("lattice,L,step", [(orc.FCC, (9, 8, 7), 1), (orc.FCC, (20, 20, 20), 53), (orc.BCC, (9, 8, 7), 1),
                                            (orc.FCC, (40, 40, 40), 997), (orc.BCC, (31, 31, 31), 211)])
def test_an_invalid_id_anywhere(lattice, L, step):
    """One invalid id, at every site in turn (whichever wavefront reads it): that
    configuration alone is NaN."""
    N, M, S = orc.n_sites(lattice, L), 5, 3
    sites = torch.arange(0, N, step, device="cuda")
    K = len(sites) + 1
    sp = torch.from_numpy(wl.iid_configs(N, M, 1, seed=5)).cuda().repeat(K, 1)
    sp[torch.arange(K - 1, device="cuda"), sites] = torch.tensor([5, 7, 8, -1, 127], dtype=torch.int8, device="cuda")[sites % 5]
    counts = torch.zeros((K, S, M, M), dtype=torch.int32, device="cuda")
    SF = torch.zeros((K, 2), dtype=torch.float64, device="cuda")
    pb.pyhea_sro_eval_batch(lattice, L, M, S, sp, counts, np.zeros((S, M, M)), np.ones(S), SF)
    torch.cuda.synchronize()
    nan = torch.isnan(SF).all(dim=1)
    assert nan[:-1].all() and not nan[-1]


def test_more_configurations_than_one_grid_holds():
    """2^24 workgroups of 256 threads are one too many for a launch."""
    lattice, L, M, S, K = orc.FCC, (3, 3, 3), 4, 1, 2**24 + 9
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    sp = torch.randint(0, M, (K, orc.n_sites(lattice, L)), dtype=torch.int8, device="cuda", generator=g)
    got = [torch.zeros((K, S, M, M), dtype=torch.int32, device="cuda") for _ in range(2)]
    pb.pyhea_sro_eval_batch(lattice, L, M, S, sp, got[0])
    pb.pyhea_tune_force_eval(1)
    try:
        pb.pyhea_sro_eval_batch(lattice, L, M, S, sp, got[1])
    finally:
        pb.pyhea_tune_force_eval(-1)
    torch.cuda.synchronize()
    assert torch.equal(got[0], got[1])
