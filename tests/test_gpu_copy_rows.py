"""Selected solutions are copied in rows of any length and number: the global
search equals the oracle where a row's bytes divide by 16, by 4 and by neither,
and where the refined solutions are more than one launch copies."""
import numpy as np
import pytest

from oracle import oracle as orc
from paper_2411_18906_amd import binding as pb

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("lattice,L,n,refine", [(orc.FCC, (3, 3, 4), 8, 5), (orc.FCC, (3, 3, 3), 7, 7),
                                                (orc.BCC, (3, 3, 3), 6, 4), (orc.FCC, (4, 4, 4), 260, 258)])
def test_search_equals_oracle(lattice, L, n, refine):
    N, M, S = orc.n_sites(lattice, L), 3, 2
    comp = [N - 2 * (N // 3), N // 3, N // 3]
    rng = np.random.default_rng(n)
    t, w = rng.uniform(-0.1, 0.1, (S, M, M)), np.ones(S)
    t = 0.5 * (t + t.transpose(0, 2, 1))
    kw = dict(n_solutions=n, iterations=2, n_refine=refine, discard_frac=0.5, seed=5, B=16, n_trials=320)
    best = torch.zeros(N, dtype=torch.int8, device="cuda")
    st, hist = pb.pyhea_global_search(lattice, L, M, S, t, w, comp, best, **kw)
    b_o, S_o, F_o, hist_o, st_o = orc.global_search(lattice, L, M, S, t, w, comp, **kw)
    np.testing.assert_array_equal(best.cpu().numpy(), b_o)
    np.testing.assert_array_equal(hist, hist_o)
    assert st["S"] == S_o and st["F"] == F_o
