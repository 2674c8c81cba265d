"""The work this library is measured on.

Each case is one pass through a public entry point as a program calls it: the
full evaluation of one configuration and of batches, trial swaps against a
fixed configuration, single Monte Carlo chains, a batch of uneven chains, the
global search, and the assignment of an external structure to lattice sites.
Sizes are those of the repository's own workloads and tests; draw() spreads
over the ranges they stand for (FCC and BCC, 2 to 6 species, 1 to 4 shells,
odd and non-cubic cells, 64 sites to 256,000 sites per configuration).
"""
from __future__ import annotations

import itertools
import math

import numpy as np
import torch

from paper_2411_18906_amd import binding as pb
from paper_2411_18906_amd import workloads as wl

FCC, BCC = wl.FCC, wl.BCC
DEVICE = "cuda"
RADII = {FCC: (2, 4, 6, 8), BCC: (3, 4, 8, 11)}          # squared, half lattice units
BASIS = {FCC: ((0, 0, 0), (1, 1, 0), (1, 0, 1), (0, 1, 1)), BCC: ((0, 0, 0), (1, 1, 1))}
WEIGHTS = (1.0, 0.5, 0.25, 0.125)


def listed():
    return [
        # a program that looks at one small cell: launches and the read-back are all there is
        dict(name="eval_one_fcc4", kind="eval_one", lattice=FCC, Lx=4, Ly=4, Lz=4, M=4, S=2),
        # the usual supercell, evaluated once (a structure just built or relaxed)
        dict(name="eval_one_fcc20", kind="eval_one", lattice=FCC, Lx=20, Ly=20, Lz=20, M=5, S=3),
        # a solution pool or a data set of the usual supercell
        dict(name="eval_batch_fcc20", kind="eval_batch", lattice=FCC, Lx=20, Ly=20, Lz=20, M=5, S=3, K=32768),
        # the large supercell, whose configuration does not fit beside others on a compute unit
        dict(name="eval_batch_fcc40", kind="eval_batch", lattice=FCC, Lx=40, Ly=40, Lz=40, M=4, S=2, K=4096),
        # an odd BCC cell: rows that no vector load divides
        dict(name="eval_batch_bcc31", kind="eval_batch", lattice=BCC, Lx=31, Ly=31, Lz=31, M=5, S=3, K=2048),
        # scoring a list of swaps against one configuration
        dict(name="trial_eval_fcc20", kind="trial_eval", lattice=FCC, Lx=20, Ly=20, Lz=20, M=5, S=3, n=4096, dN=True),
        # the smallest search: 10^4 trials on 256 sites, with its accepted-swap log
        dict(name="chain_fcc4", kind="chain", lattice=FCC, Lx=4, Ly=4, Lz=4, M=4, S=2, T=10**4, B=64, mode=0,
             tau=0.0, zero_target=True, log=1024),
        # the usual search: 10^6 trials on 32,000 sites, random solid solution wanted
        dict(name="chain_fcc20", kind="chain", lattice=FCC, Lx=20, Ly=20, Lz=20, M=5, S=3, T=10**6, B=64, mode=0,
             tau=0.0, zero_target=True, log=0),
        # the large search: 10^7 trials on 256,000 sites towards a given SRO
        dict(name="chain_fcc40", kind="chain", lattice=FCC, Lx=40, Ly=40, Lz=40, M=4, S=2, T=10**7, B=64, mode=0,
             tau=0.0, zero_target=False, log=0),
        # many uneven searches at once
        dict(name="chains_512", kind="chains", n=512, T=10**5, mix=4),
        # the whole workflow towards a given SRO: random pools, evaluation, refinement (the paper's
        # performance preset: 64 solutions, 6 iterations, 64 tasks, depth 8)
        dict(name="global_fcc20", kind="global", lattice=FCC, Lx=20, Ly=20, Lz=20, M=5, S=3, pool=64, iterations=6,
             refine=32, discard=0.5, T=10**5, B=64, depth=8),
        # reading a structure of another code back onto the lattice
        dict(name="map_fcc40", kind="map", lattice=FCC, Lx=40, Ly=40, Lz=40, M=4),
    ]


def _L(case):
    return (case["Lx"], case["Ly"], case["Lz"])


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _cell(rng, lattice, n_lo, n_hi):
    """A cubic or slightly uneven cell of about n sites, at least 3 cells wide."""
    base = (_log_uniform(rng, n_lo, n_hi) / wl.BASIS_PER_CELL[lattice]) ** (1.0 / 3.0)
    if rng.random() < 0.5:
        c = max(3, round(base))
        return dict(Lx=c, Ly=c, Lz=c)
    while True:
        L = tuple(max(3, round(base * rng.uniform(0.75, 1.3))) for _ in range(3))
        if pb.n_sites(lattice, L) <= n_hi:
            return dict(Lx=L[0], Ly=L[1], Lz=L[2])


def draw(rng):
    kind = rng.choice(["eval_one", "eval_batch", "eval_batch", "eval_batch", "trial_eval", "chain", "chain",
                       "chains", "global", "map"])
    lattice = rng.choice([FCC, BCC])
    M = rng.choice([2, 3, 4, 4, 5, 5, 6])
    S = rng.choice([1, 2, 2, 3, 3, 4])
    if kind == "eval_one":
        return dict(kind=kind, lattice=lattice, **_cell(rng, lattice, 128, 256000), M=M, S=S)
    if kind == "eval_batch":
        cell = _cell(rng, lattice, 256, 256000)
        sites = _log_uniform(rng, 10**6, 10**9)
        K = min(60000, max(1, int(sites / pb.n_sites(lattice, _L(cell)))))
        return dict(kind=kind, lattice=lattice, **cell, M=M, S=S, K=K)
    if kind == "trial_eval":
        return dict(kind=kind, lattice=lattice, **_cell(rng, lattice, 256, 256000), M=M, S=S,
                    n=int(_log_uniform(rng, 64, 65536)), dN=rng.random() < 0.5)
    if kind == "chain":
        return dict(kind=kind, lattice=lattice, **_cell(rng, lattice, 256, 256000), M=M, S=min(S, 3),
                    T=int(_log_uniform(rng, 10**4, 10**6)), B=rng.choice([32, 64, 64, 100, 256]),
                    mode=rng.choice([0, 0, 0, 1]), tau=0.0, zero_target=rng.random() < 0.4, log=0)
    if kind == "chains":
        return dict(kind=kind, n=int(_log_uniform(rng, 4, 512)), T=int(_log_uniform(rng, 10**3, 10**5)),
                    mix=rng.randrange(1000))
    if kind == "global":
        pool = int(_log_uniform(rng, 8, 64))
        return dict(kind=kind, lattice=lattice, **_cell(rng, lattice, 256, 32000), M=min(M, 5), S=min(S, 3), pool=pool,
                    iterations=rng.randint(2, 6), refine=max(1, pool // 2), discard=0.5, T=10**5, B=64,
                    depth=rng.choice([4, 8, 16]), zero_target=rng.random() < 0.4)
    return dict(kind="map", lattice=lattice, **_cell(rng, lattice, 256, 256000), M=M)


# --------------------------------------------------------------------------- inputs

def _composition(N, M):
    return wl.largest_remainder(N, np.ones(M))


def _objective(case, seed):
    """Targets reachable by the composition (per shell, sum_j c_j alpha_ij = 0), or 0."""
    M, S = case["M"], case["S"]
    if case.get("zero_target", False):
        return np.zeros((S, M, M)), np.ones(S)
    n = _composition(pb.n_sites(case["lattice"], _L(case)), M)
    return wl.projected_target(S, M, n / n.sum(), seed), np.array(WEIGHTS[:S])


def _generator(seed):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(seed)
    return g


def _species(case, seed):
    N = pb.n_sites(case["lattice"], _L(case))
    return torch.from_numpy(wl.shuffled_config(N, _composition(N, case["M"]), seed, 0)).to(DEVICE)


def _batch_species(case, seed):
    """K independent uniform arrangements (the first M sites hold every species once)."""
    N, M = pb.n_sites(case["lattice"], _L(case)), case["M"]
    sp = torch.randint(0, M, (case["K"], N), dtype=torch.int8, device=DEVICE, generator=_generator(seed))
    sp[:, :M] = torch.arange(M, dtype=torch.int8, device=DEVICE)
    return sp


def _pairs(case, seed):
    N = pb.n_sites(case["lattice"], _L(case))
    return torch.randint(0, N, (case["n"], 2), dtype=torch.int32, device=DEVICE, generator=_generator(seed + 1))


def _site_positions(lattice, L):
    """[N][3] half-unit positions of the sites in site order."""
    z, y, x = np.meshgrid(*(np.arange(L[a]) for a in (2, 1, 0)), indexing="ij")
    cells = np.stack([x, y, z], axis=-1).reshape(-1, 1, 3)
    return (2 * cells + np.array(BASIS[lattice]).reshape(1, -1, 3)).reshape(-1, 3)


def _structure(case, seed):
    """A relaxed structure of another code: sites displaced by thermal vibration,
    atoms in a random order, any periodic image, a slightly stretched box."""
    rng = np.random.default_rng(seed)
    lattice, L = case["lattice"], _L(case)
    N = pb.n_sites(lattice, L)
    box = np.array(L) * 3.6 * (1.0 + 0.01 * rng.uniform(-1.0, 1.0, 3))
    pos = _site_positions(lattice, L) * (box / (2.0 * np.array(L)))
    pos += np.clip(rng.normal(0.0, 0.08, (N, 3)), -0.3, 0.3)
    pos += rng.integers(-1, 2, (N, 3)) * box
    species = wl.shuffled_config(N, _composition(N, case["M"]), seed, 0)
    order = rng.permutation(N)
    return box, pos[order], species[order], species, order


def prepare(case, seed):
    kind = case["kind"]
    if kind == "chains":
        chains = wl.mixed_chains(n_chains=case["n"], seed=case["mix"], n_trials=case["T"])
        for c in chains:   # the cells and compositions are the case's, the arrangements and targets the seed's
            n = np.bincount(c.species, minlength=c.M)
            c.species = wl.shuffled_config(c.N, n, seed, c.chain_id)
            c.target = wl.projected_target(c.S, c.M, n / c.N, seed, stream=c.chain_id + 1000)
            c.seed = seed
        sp = torch.from_numpy(np.concatenate([c.species for c in chains])).to(DEVICE)
        return dict(kind=kind, initial=sp, offsets=np.concatenate([[0], np.cumsum([c.N for c in chains])]),
                    pack=pb.pack_batch([(c.lattice, c.L, c.M, c.S, c.target, c.weight) for c in chains],
                                       [pb.make_params(c.seed, c.chain_id, c.n_trials, c.B) for c in chains]))
    st = dict(kind=kind, lattice=case["lattice"], L=_L(case), M=case["M"])
    if kind == "map":
        box, xyz, types, _, _ = _structure(case, seed)
        N = len(types)
        st.update(box=box, xyz=torch.from_numpy(xyz).to(DEVICE), types=torch.from_numpy(types).to(DEVICE),
                  species=torch.empty(N, dtype=torch.int8, device=DEVICE),
                  atom=torch.empty(N, dtype=torch.int32, device=DEVICE))
        return st
    M, S = case["M"], case["S"]
    st["S"] = S
    st["target"], st["weight"] = _objective(case, seed)
    if kind == "eval_one":
        st["species"] = _species(case, seed)
    elif kind == "eval_batch":
        st.update(species=_batch_species(case, seed),
                  counts=torch.empty((case["K"], S, M, M), dtype=torch.int32, device=DEVICE),
                  S_F=torch.empty((case["K"], 2), dtype=torch.float64, device=DEVICE))
    elif kind == "trial_eval":
        st.update(species=_species(case, seed), pairs=_pairs(case, seed),
                  dS=torch.empty(case["n"], dtype=torch.float64, device=DEVICE),
                  dN=torch.empty((case["n"], S, M, M), dtype=torch.int32, device=DEVICE) if case["dN"] else None)
    elif kind == "chain":
        st.update(initial=_species(case, seed),
                  params=pb.make_params(seed, 0, case["T"], case["B"], case["mode"], 0, case["tau"]),
                  log=torch.zeros((case["log"], 4), dtype=torch.int32, device=DEVICE) if case["log"] else None)
    else:
        N = pb.n_sites(case["lattice"], _L(case))
        st.update(composition=_composition(N, M), best=torch.empty(N, dtype=torch.int8, device=DEVICE), seed=seed,
                  search={k: case[k] for k in ("pool", "iterations", "refine", "discard", "T", "B", "depth")})
    return st


def _chain_numbers(st):
    return {k: np.ascontiguousarray(st[k]) if isinstance(st, np.ndarray) else st[k]
            for k in ("trials", "null_trials", "commits", "steps", "S", "F")}


def run(state):
    s = state
    if s["kind"] == "eval_one":
        counts, alpha, S, F = pb.pyhea_sro_eval(s["lattice"], s["L"], s["M"], s["S"], s["species"], s["target"],
                                                s["weight"])
        return dict(counts=counts, alpha=alpha, S=S, F=F)
    if s["kind"] == "eval_batch":
        pb.pyhea_sro_eval_batch(s["lattice"], s["L"], s["M"], s["S"], s["species"], s["counts"], s["target"],
                                s["weight"], s["S_F"])
        return dict(counts=s["counts"], S_F=s["S_F"])
    if s["kind"] == "trial_eval":
        pb.pyhea_trial_eval(s["lattice"], s["L"], s["M"], s["S"], s["species"], s["target"], s["weight"], s["pairs"],
                            s["dS"], s["dN"])
        return dict(dS=s["dS"]) if s["dN"] is None else dict(dS=s["dS"], dN=s["dN"])
    if s["kind"] == "chain":
        sp = s["initial"].clone()
        st, counts = pb.pyhea_mc_run(s["lattice"], s["L"], s["M"], s["S"], s["target"], s["weight"], sp, s["params"],
                                     s["log"])
        out = dict(species=sp, counts=counts, **_chain_numbers(st))
        return out if s["log"] is None else dict(out, log=s["log"])
    if s["kind"] == "chains":
        sp = s["initial"].clone()
        st = pb.pyhea_mc_batch(s["pack"], sp, s["offsets"])
        return dict(species=sp, **_chain_numbers(st))
    if s["kind"] == "global":
        g = s["search"]
        st, hist = pb.pyhea_global_search(s["lattice"], s["L"], s["M"], s["S"], s["target"], s["weight"],
                                          s["composition"], s["best"], n_solutions=g["pool"],
                                          iterations=g["iterations"], n_refine=g["refine"], discard_frac=g["discard"],
                                          seed=s["seed"], B=g["B"], n_trials=g["T"], depth_limit=g["depth"])
        return dict(best=s["best"], history=hist, **st)
    pb.pyhea_map_sites(s["lattice"], s["L"], s["M"], 1, s["box"], 1.2, s["xyz"], s["types"], s["species"], s["atom"])
    return dict(species=s["species"], atom=s["atom"])


def work(case):
    """Bytes: each input read and each output written once.  Operations: two per
    pair of an evaluation (a pair is classified and counted once), and per trial
    the draw, the 2 (1 + Z) species looked at and the changed rows of the
    objective (about 6 operations per entry)."""
    if case["kind"] == "chains":
        sites = 3800 * case["n"]   # the mean of a log-uniform size in 250 .. 16,000
        return dict(bytes=2 * sites, flops=case["n"] * case["T"] * (2 * 18 + 2 * 2 * 4.5 * 6))
    N = pb.n_sites(case["lattice"], _L(case))
    if case["kind"] == "map":
        return dict(bytes=N * (24 + 1 + 1 + 4), flops=30 * N)
    M, S = case["M"], case["S"]
    Z = len(_offsets(case["lattice"], S))
    E = S * M * M
    if case["kind"] == "eval_one":
        return dict(bytes=N + 20 * E, flops=N * Z)
    if case["kind"] == "eval_batch":
        return dict(bytes=case["K"] * (N + 4 * E + 16), flops=case["K"] * N * Z)
    trial = 2 * (1 + Z) + 2 * S * M * 6
    if case["kind"] == "trial_eval":
        return dict(bytes=N + case["n"] * (8 + 8 + (4 * E if case["dN"] else 0)), flops=N * Z + case["n"] * trial)
    if case["kind"] == "chain":
        return dict(bytes=2 * N + 8 * E, flops=2 * N * Z + case["T"] * trial)
    pool = case["pool"] * case["iterations"]
    # a refinement runs a few tens of steps before its depth limit ends it
    return dict(bytes=pool * N * 2, flops=pool * N * Z + case["refine"] * case["iterations"] * 2000 * trial)


# --------------------------------------------------------------------------- plain 64-bit values

def _offsets(lattice, S):
    """(shell, (dx, dy, dz)) of every neighbour vector of shells 1..S, half units."""
    out = []
    for d in itertools.product(range(-3, 4), repeat=3):
        on = sum(d) % 2 == 0 if lattice == FCC else len({v % 2 for v in d}) == 1
        r2 = sum(v * v for v in d)
        if on and r2 in RADII[lattice][:S]:
            out.append((RADII[lattice].index(r2), d))
    return sorted(out)


def _pair_counts(lattice, L, M, S, species):
    """Ordered pair counts [K][S][M][M] int64 of species [K][N]."""
    A = wl.BASIS_PER_CELL[lattice]
    out = torch.zeros((species.shape[0], S, M, M), dtype=torch.int64, device=species.device)
    step = max(1, (1 << 26) // species.shape[1])
    for c0 in range(0, species.shape[0], step):
        cells = species[c0:c0 + step].reshape(-1, L[2], L[1], L[0], A)
        planes = [cells[..., b].contiguous() for b in range(A)]
        res = out[c0:c0 + step]
        for b, base in enumerate(BASIS[lattice]):
            for k, d in _offsets(lattice, S):
                if d < tuple(-v for v in d):
                    continue                       # one of each +-d pair; the other is the transpose
                to = [base[a] + d[a] for a in range(3)]
                b2 = BASIS[lattice].index(tuple(v % 2 for v in to))
                sh = [(to[a] - BASIS[lattice][b2][a]) // 2 for a in range(3)]
                nb = torch.roll(planes[b2], shifts=(-sh[2], -sh[1], -sh[0]), dims=(1, 2, 3))
                code = (planes[b] * M + nb).reshape(cells.shape[0], -1)
                for i in range(M):
                    for j in range(M):
                        n = (code == i * M + j).sum(dim=1)
                        res[:, k, i, j] += n
                        res[:, k, j, i] += n
    return out


def _alpha_objective(lattice, M, N, counts, target, weight):
    """alpha, S and F in binary64 from counts [K][S][M][M]."""
    c = counts.double()
    z = torch.tensor([sum(1 for k, _ in _offsets(lattice, counts.shape[1]) if k == s) for s in range(counts.shape[1])],
                     dtype=torch.float64, device=c.device)
    n = c[:, 0].sum(dim=2) / z[0]
    alpha = 1.0 - c * N / (n[:, None, :, None] * n[:, None, None, :] * z[None, :, None, None])
    t = torch.as_tensor(target, dtype=torch.float64, device=c.device)
    w = torch.as_tensor(weight, dtype=torch.float64, device=c.device)
    S = (((alpha - t) ** 2).sum(dim=(2, 3)) * w).sum(dim=1)
    return alpha, S, S.sqrt()


def _exact_trials(case, seed):
    lattice, L, M, S = case["lattice"], _L(case), case["M"], case["S"]
    N = pb.n_sites(lattice, L)
    sp = _species(case, seed)
    pairs = _pairs(case, seed).long()
    target, weight = _objective(case, seed)
    counts = _pair_counts(lattice, L, M, S, sp.reshape(1, N))
    _, s0, _ = _alpha_objective(lattice, M, N, counts, target, weight)
    pos = torch.from_numpy(_site_positions(lattice, L)).to(DEVICE)
    box = torch.tensor([2 * v for v in L], device=DEVICE)
    site_at = torch.full((2 * L[2], 2 * L[1], 2 * L[0]), -1, dtype=torch.int64, device=DEVICE)
    site_at[pos[:, 2], pos[:, 1], pos[:, 0]] = torch.arange(N, device=DEVICE)
    p, q = pairs[:, 0], pairs[:, 1]
    a, b = sp[p].long(), sp[q].long()
    n = len(p)
    rows = torch.arange(n, device=DEVICE)
    dN = torch.zeros((n, S, M, M), dtype=torch.int64, device=DEVICE)
    for k, d in _offsets(lattice, S):
        off = torch.tensor(d, device=DEVICE)
        for site, partner, old, new in ((p, q, a, b), (q, p, b, a)):
            r = (pos[site] + off) % box
            r = site_at[r[:, 2], r[:, 1], r[:, 0]]
            # the ordered pairs (site, r) and (r, site); the pair of the two swapped
            # sites keeps its species
            other = sp[r].long()
            one = (r != partner).long()
            for i, j, v in ((old, other, -one), (new, other, one)):
                dN.index_put_((rows, torch.full_like(r, k), i, j), v, accumulate=True)
                dN.index_put_((rows, torch.full_like(r, k), j, i), v, accumulate=True)
    # each term's change as d1^2 - d0^2 = (a1 - a0)(a1 + a0 - 2 t)
    c = counts.double()
    z = [sum(1 for kk, _ in _offsets(lattice, S) if kk == s) for s in range(S)]
    tot = c[0, 0].sum(dim=1) / z[0]
    z = torch.tensor(z, dtype=torch.float64, device=DEVICE)
    R = N / (tot[None, :, None] * tot[None, None, :] * z[:, None, None])
    t = torch.as_tensor(target, dtype=torch.float64, device=DEVICE)
    w = torch.as_tensor(weight, dtype=torch.float64, device=DEVICE)
    a0 = 1.0 - c[0] * R
    da = -dN.double() * R
    dS = ((da * (da + 2.0 * (a0 - t))).sum(dim=(2, 3)) * w).sum(dim=1)
    return dict(dS=dS, dN=dN.int()) if case["dN"] else dict(dS=dS)


def exact(case, seed):
    kind = case["kind"]
    if kind == "eval_one":
        N = pb.n_sites(case["lattice"], _L(case))
        target, weight = _objective(case, seed)
        c = _pair_counts(case["lattice"], _L(case), case["M"], case["S"], _species(case, seed).reshape(1, N))
        alpha, S, F = _alpha_objective(case["lattice"], case["M"], N, c, target, weight)
        return dict(counts=c[0].cpu().numpy(), alpha=alpha[0].cpu().numpy(), S=float(S[0]), F=float(F[0]))
    if kind == "eval_batch":
        N = pb.n_sites(case["lattice"], _L(case))
        target, weight = _objective(case, seed)
        c = _pair_counts(case["lattice"], _L(case), case["M"], case["S"], _batch_species(case, seed))
        _, S, F = _alpha_objective(case["lattice"], case["M"], N, c, target, weight)
        return dict(counts=c.int(), S_F=torch.stack([S, F], dim=1))
    if kind == "trial_eval":
        return _exact_trials(case, seed)
    if kind == "map":
        _, _, _, species, order = _structure(case, seed)
        atom = np.empty(len(order), np.int32)
        atom[order] = np.arange(len(order), dtype=np.int32)
        return dict(species=torch.from_numpy(species).to(DEVICE), atom=torch.from_numpy(atom).to(DEVICE))
    # a chain's outcome is a trajectory of accepted swaps, one trial after another:
    # no plain array expression gives it
    return None
