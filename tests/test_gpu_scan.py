"""Quiet chains: once a chain commits rarely, its next steps are evaluated by
the whole chip in windows and the chain goes on at the first step that commits.
Every trajectory must be the oracle's: accepted-swap log, final configuration,
counters (the null draws of scanned steps among them), S and the maintained
counts, for every store, both commit modes, one and several slot groups per
step, cells two cells wide, a depth limit reached inside a window, a partial
last step and several chains in one call."""
import numpy as np
import pytest

from oracle import oracle as orc
from paper_2411_18906_amd import binding as pb
from paper_2411_18906_amd import workloads as wl

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _problem(lattice, L, M, S, seed, zero):
    N = pb.n_sites(lattice, L)
    n = wl.largest_remainder(N, np.ones(M))
    sp = wl.shuffled_config(N, n, seed, 0)
    tgt = np.zeros((S, M, M)) if zero else wl.projected_target(S, M, n / N, seed)
    return sp, tgt, np.array([1.0, 0.5, 0.25, 0.125][:S])


# lattice, L, M, S, T, B, mode, depth, tau, zero target, launch variant
CASES = [
    (wl.FCC, (4, 4, 4), 4, 2, 30011, 64, 0, 0, 0.0, True, -1),       # LDS bytes, partial last step
    (wl.FCC, (4, 4, 4), 4, 2, 30000, 64, 0, 0, 0.0, True, 1),        # LDS nibbles
    (wl.FCC, (4, 4, 4), 4, 2, 30000, 64, 0, 0, 0.0, True, 2),        # HBM
    (wl.BCC, (2, 5, 6), 3, 3, 40000, 100, 0, 0, 0.0, False, -1),     # two cells wide, two slot groups
    (wl.BCC, (7, 6, 5), 5, 4, 60000, 256, 0, 0, 0.0, False, -1),     # halo of two, four slot groups
    (wl.FCC, (6, 5, 4), 7, 3, 40000, 33, 1, 0, 0.0, False, -1),      # BEST, wide histograms
    (wl.FCC, (5, 5, 5), 5, 3, 10**6, 64, 0, 60, 0.0, True, -1),      # depth limit inside a window
    (wl.FCC, (5, 5, 5), 5, 3, 10**6, 64, 0, 1000, 1e-9, True, -1),   # and past several commits, margin tau
    (wl.FCC, (8, 8, 8), 4, 2, 300000, 64, 0, 0, 0.0, False, -1),     # many rounds
]


@pytest.mark.parametrize("case", CASES)
def test_quiet_chain_equals_oracle(case):
    lattice, L, M, S, T, B, mode, depth, tau, zero, variant = case
    sp, tgt, w = _problem(lattice, L, M, S, 17, zero)
    ref = orc.mc_run(lattice, L, M, S, tgt, w, sp, seed=5, chain_id=3, n_trials=T, B=B, mode=mode, depth_limit=depth,
                     tau=tau)
    sp_o, log_o, st_o, cnt_o = ref
    pb.pyhea_tune_force(variant)
    try:
        for _ in range(3):   # eager, recorded, replayed
            d = torch.from_numpy(sp).cuda()
            log = torch.zeros((1 << 14, 4), dtype=torch.int32, device="cuda")
            st, cnt = pb.pyhea_mc_run(lattice, L, M, S, tgt, w, d, pb.make_params(5, 3, T, B, mode, depth, tau), log)
            np.testing.assert_array_equal(d.cpu().numpy(), sp_o)
            np.testing.assert_array_equal(cnt, cnt_o)
            n = st["log_len"]
            np.testing.assert_array_equal(log[:n].cpu().numpy().view(np.uint32), np.asarray(log_o)[:n])
            for k in ("trials", "null_trials", "commits", "steps", "stop_reason", "S"):
                assert st[k] == st_o[k], k
            torch.cuda.synchronize()
    finally:
        pb.pyhea_tune_force(-1)


def test_several_chains_in_one_call():
    chains = wl.mixed_chains(n_chains=9, seed=77, n_trials=40000)
    chains[4].n_trials = 500      # too short to scan, in a call that does
    chains[6].n_trials = 0
    species = np.concatenate([c.species for c in chains])
    off = np.concatenate([[0], np.cumsum([c.N for c in chains])])
    pars = [pb.make_params(c.seed, c.chain_id, c.n_trials, c.B) for c in chains]
    probs = [(c.lattice, c.L, c.M, c.S, c.target, c.weight) for c in chains]
    for _ in range(3):
        d = torch.from_numpy(species).cuda()
        stats = pb.pyhea_mc_batch(probs, d, off, pars)
        fin = d.cpu().numpy()
        for i, c in enumerate(chains):
            sp_o, _, st_o, _ = orc.mc_run(c.lattice, c.L, c.M, c.S, c.target, c.weight, c.species, seed=c.seed,
                                          chain_id=c.chain_id, n_trials=c.n_trials, B=c.B)
            np.testing.assert_array_equal(fin[off[i]:off[i + 1]], sp_o, err_msg=f"chain {i}")
            for k in ("trials", "null_trials", "commits", "steps", "S"):
                assert stats[i][k] == st_o[k], (i, k)


@pytest.fixture
def eager():
    """No recorded graphs: a process keeps the first 32 structures that are called twice."""
    pb.pyhea_tune_graphs(False)
    yield
    pb.pyhea_tune_graphs(True)


@pytest.mark.parametrize("depth", [4, 63, 64, 79, 80, 81, 120])
def test_depth_limit_around_the_first_scan(depth, eager):
    """A single chain scans from a depth limit of 80 on."""
    test_quiet_chain_equals_oracle((wl.FCC, (5, 5, 5), 5, 3, 10**6, 64, 0, depth, 0.0, True, -1))
    test_quiet_chain_equals_oracle((wl.BCC, (6, 5, 4), 4, 2, 10**6, 100, 0, depth, 0.0, False, -1))


@pytest.mark.parametrize("n,steps", [(1, 223), (1, 224), (2, 749), (2, 750), (16, 1519), (16, 1520), (17, 3000)])
@pytest.mark.parametrize("depth", [0, 99, 100, 380])
def test_calls_around_the_least_steps(n, steps, depth):
    """The least steps and depth limit of a call that scans grow with its chains."""
    lattice, L, M, S, B = wl.FCC, (3, 4, 3), 4, 2, 32
    jobs = [_problem(lattice, L, M, S, 30 + i, False) for i in range(n)]
    N = len(jobs[0][0])
    pars = [pb.make_params(9, i, steps * B if i == 0 else 50 * B, B, 0, depth, 0.0) for i in range(n)]
    d = torch.from_numpy(np.concatenate([j[0] for j in jobs])).cuda()
    stats = pb.pyhea_mc_batch([(lattice, L, M, S, j[1], j[2]) for j in jobs], d, np.arange(n + 1) * N, pars)
    fin = d.cpu().numpy()
    for i in range(min(n, 3)):
        sp, tgt, w = jobs[i]
        sp_o, _, st_o, _ = orc.mc_run(lattice, L, M, S, tgt, w, sp, seed=9, chain_id=i,
                                      n_trials=(steps if i == 0 else 50) * B, B=B, depth_limit=depth)
        np.testing.assert_array_equal(fin[i * N:(i + 1) * N], sp_o)
        for k in ("trials", "null_trials", "commits", "steps", "S"):
            assert stats[i][k] == st_o[k], (i, k)


@pytest.mark.parametrize("B", [1, 3, 15, 16])
@pytest.mark.parametrize("lattice,L,M,S,variant", [(wl.FCC, (4, 4, 4), 4, 2, -1), (wl.FCC, (3, 4, 5), 7, 3, 1),
                                                   (wl.BCC, (6, 5, 4), 3, 4, 2)])
def test_few_candidates_a_step(lattice, L, M, S, variant, B, eager):
    """Below 16 candidates a step windows open after quiet steps only."""
    for mode, depth, tau in ((0, 0, 0.0), (1, 0, 0.0), (0, 13, 0.0), (0, 0, -1e-6)):
        test_quiet_chain_equals_oracle((lattice, L, M, S, 700 * B + B // 2, B, mode, depth, tau, False, variant))
