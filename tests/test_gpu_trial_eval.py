"""Trial swaps by half wavefronts: dS and dN equal to the oracle where the split
can go wrong -- one pair to more pairs than a launch's groups, a last workgroup
partly filled, cells so small that a site's neighbours repeat or are the other
site, all numbers of species and shells -- and nothing is written for a
configuration that is refused."""
import numpy as np
import pytest

from oracle import oracle as orc
from paper_2411_18906_amd import binding as pb
from paper_2411_18906_amd import workloads as wl

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("lattice,L,M,S,n", [
    (orc.FCC, (3, 3, 3), 8, 4, 1), (orc.FCC, (3, 4, 5), 2, 1, 7), (orc.BCC, (3, 3, 3), 8, 4, 9),
    (orc.FCC, (4, 4, 4), 5, 3, 8), (orc.BCC, (5, 4, 3), 3, 2, 33), (orc.FCC, (6, 5, 4), 4, 4, 17),
    (orc.FCC, (20, 20, 20), 5, 3, 40001),
])
def test_pairs_equal_oracle(lattice, L, M, S, n):
    N = orc.n_sites(lattice, L)
    sp = wl.iid_configs(N, M, 1, seed=M)[0]
    sp[:M] = np.arange(M)
    rng = np.random.default_rng(n)
    tgt, w = rng.uniform(-0.2, 0.2, (S, M, M)), rng.uniform(0.1, 1.0, S)
    pairs = rng.integers(0, N, size=(n, 2)).astype(np.int32)
    if n > 8:
        pairs[3] = pairs[3, 0]              # a site with itself
        pairs[4] = [0, 1]                   # neighbours
        pairs[5] = [-1, 0]
        pairs[6] = [0, N]
    dS = torch.full((n,), 7.0, dtype=torch.float64, device="cuda")
    dN = torch.full((n, S, M, M), 7, dtype=torch.int32, device="cuda")
    pb.pyhea_trial_eval(lattice, L, M, S, torch.from_numpy(sp).cuda(), tgt, w, torch.from_numpy(pairs).cuda(), dS, dN)
    dS2 = torch.zeros_like(dS)
    pb.pyhea_trial_eval(lattice, L, M, S, torch.from_numpy(sp).cuda(), tgt, w, torch.from_numpy(pairs).cuda(), dS2)
    ds, dn = dS.cpu().numpy(), dN.cpu().numpy()
    np.testing.assert_array_equal(ds, dS2.cpu().numpy())
    which = range(n) if n < 100 else list(range(10)) + list(range(10, n, n // 60)) + [n - 1]
    for u in which:
        p, q = int(pairs[u, 0]), int(pairs[u, 1])
        if p < 0 or q >= N:
            assert np.isnan(ds[u]) and (dn[u] == 7).all()
            continue
        np.testing.assert_array_equal(dn[u], orc.swap_delta(lattice, L, M, S, sp, p, q))
        assert ds[u] == orc.swap_dS(lattice, L, M, S, sp, p, q, tgt, w)


@pytest.mark.parametrize("n", [0, 20])
@pytest.mark.parametrize("value", [4, -1, 0])
def test_refused_configuration_writes_nothing(n, value):
    N, M, S = orc.n_sites(orc.FCC, (4, 4, 4)), 4, 2
    sp = wl.iid_configs(N, M, 1, seed=1)[0]
    if value == 0:
        sp[sp == 3] = 0                     # a species is absent
    else:
        sp[N - 1] = value
    pairs = torch.from_numpy(np.random.default_rng(0).integers(0, N, size=(n, 2)).astype(np.int32)).cuda()
    dS = torch.full((n,), 7.0, dtype=torch.float64, device="cuda")
    dN = torch.full((n, S, M, M), 7, dtype=torch.int32, device="cuda")
    with pytest.raises(pb.PyheaError):
        pb.pyhea_trial_eval(orc.FCC, (4, 4, 4), M, S, torch.from_numpy(sp).cuda(), np.zeros((S, M, M)), np.ones(S),
                            pairs, dS, dN)
    assert (dS == 7).all() and (dN == 7).all()


@pytest.mark.parametrize("lattice,L,M,S", [
    (orc.FCC, (3, 3, 3), 8, 4), (orc.FCC, (2, 2, 3), 2, 2), (orc.BCC, (3, 3, 3), 7, 4), (orc.FCC, (4, 4, 4), 5, 3),
    (orc.BCC, (5, 4, 3), 3, 2), (orc.FCC, (6, 5, 4), 4, 1), (orc.FCC, (20, 20, 20), 6, 3),
])
@pytest.mark.parametrize("n,with_dN", [(80000, False), (80037, False), (200000, True), (200191, True), (600001, True)])
def test_many_pairs_equal_few(lattice, L, M, S, n, with_dN):
    """From 80,000 pairs (200,000 with dN) a lane takes a pair: the results of calls with fewer."""
    N = orc.n_sites(lattice, L)
    sp = wl.iid_configs(N, M, 1, seed=M)[0]
    sp[:M] = np.arange(M)
    sp = torch.from_numpy(sp).cuda()
    rng = np.random.default_rng(n)
    tgt, w = rng.uniform(-0.2, 0.2, (S, M, M)), rng.uniform(0.1, 1.0, S)
    pairs = rng.integers(0, N, size=(n, 2)).astype(np.int32)
    pairs[3::1000, 1] = pairs[3::1000, 0]    # a site with itself
    pairs[4::1000] = [0, 1]                  # neighbours
    pairs[5::1000] = [-1, 0]
    pairs[n - 1] = [0, N]
    pairs = torch.from_numpy(pairs).cuda()

    def call(pairs, guard):
        dS = torch.full((len(pairs) + guard,), 7.0, dtype=torch.float64, device="cuda")
        dN = torch.full((len(pairs) + guard, S, M, M), 7, dtype=torch.int32, device="cuda")
        pb.pyhea_trial_eval(lattice, L, M, S, sp, tgt, w, pairs, dS[:len(pairs)], dN[:len(pairs)] if with_dN else None)
        assert (dS[len(pairs):] == 7).all() and (dN[len(pairs):] == 7).all()
        return dS[:len(pairs)], dN[:len(pairs)]

    dS, dN = call(pairs, 300)
    few = [call(p, 0) for p in pairs.split(50000)]
    want_S, want_N = torch.cat([f[0] for f in few]), torch.cat([f[1] for f in few])
    assert torch.equal(dS.view(torch.int64), want_S.view(torch.int64)) and torch.equal(dN, want_N)
    assert torch.isnan(dS[5::1000]).all() and torch.isnan(dS[n - 1])
