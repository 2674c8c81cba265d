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
