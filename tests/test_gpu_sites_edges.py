"""Nearest-site assignment where a position lies on or beside a face of the box
(the decoded coordinate is then -1 .. 2 L + 1 and wraps once), in boxes of one
cell, and with far, unknown and doubled atoms in several workgroups at once."""
import numpy as np
import pytest

from oracle import oracle as orc
from paper_2411_18906_amd import binding as pb
import sites_inputs as si

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("eps", [0.0, -1e-13, 1e-13, -0.2, 0.2])
@pytest.mark.parametrize("lattice,L", [(orc.FCC, (1, 1, 1)), (orc.BCC, (1, 1, 1)), (orc.FCC, (1, 2, 3)),
                                       (orc.BCC, (3, 2, 1)), (orc.FCC, (9, 8, 7))])
def test_positions_beside_the_faces(lattice, L, eps):
    N, M, box = orc.n_sites(lattice, L), 3, tuple(4.0 * v for v in L)
    sp = (np.arange(N) % M).astype(np.int8)
    xyz, types, _ = si.structure(lattice, L, box, sp, 0.0, seed=1, images=True, shuffle=True)
    xyz = xyz + eps
    out = torch.zeros(N, dtype=torch.int8, device="cuda")
    owner = torch.zeros(N, dtype=torch.int32, device="cuda")
    pb.pyhea_map_sites(lattice, L, M, 1, box, 0.9, torch.from_numpy(xyz).cuda(), torch.from_numpy(types).cuda(), out, owner)
    sp_o, site_o = orc.map_sites(lattice, L, M, box, 0.9, xyz, types)
    np.testing.assert_array_equal(out.cpu().numpy(), sp_o)
    np.testing.assert_array_equal(owner.cpu().numpy()[site_o], np.arange(N))


@pytest.mark.parametrize("fault,match", [("far", "farther than max_disp"), ("nan", "farther than max_disp"),
                                         ("type", "types must lie"), ("double", "two atoms")])
def test_many_faults_at_once(fault, match):
    lattice, L, box, M = orc.FCC, (10, 10, 10), (40.0, 40.0, 40.0), 2
    N = orc.n_sites(lattice, L)
    sp = (np.arange(N) % M).astype(np.int8)
    xyz, types, _ = si.structure(lattice, L, box, sp, 0.0, seed=2, images=False, shuffle=False)
    which = np.arange(3, N, 7)
    if fault == "far":
        xyz[which, 1] += 0.9
    elif fault == "nan":
        xyz[which, 2] = np.nan
    elif fault == "type":
        types[which] = -1
    else:
        xyz[which] = xyz[which - 1]
    out = torch.zeros(N, dtype=torch.int8, device="cuda")
    with pytest.raises(pb.PyheaError, match=match):
        pb.pyhea_map_sites(lattice, L, M, 1, box, 0.5, torch.from_numpy(xyz).cuda(), torch.from_numpy(types).cuda(), out)


def residual(x, L, box):
    """The kernel's reduction into the box (half lattice units), in the same binary64 steps."""
    period = 2.0 * L
    v = x * (2.0 * L / box)
    return v - period * np.floor(v / period)


@pytest.mark.parametrize("lattice,L,box", [(orc.FCC, (10, 10, 10), 40.0), (orc.BCC, (10, 10, 10), 40.0),
                                           (orc.FCC, (40, 7, 5), 144.0)])
def test_coordinates_of_any_size(lattice, L, box):
    """Beyond 2^53 periods the reduction leaves residuals far outside the box; the site is
    then the residual's modulo the box, and nothing outside the buffers is written."""
    N, M, m = orc.n_sites(lattice, L), 3, 2 * L[0]
    boxes = (box, 4.0 * L[1], 4.0 * L[2])
    sp = (np.arange(N) % M).astype(np.int8)
    xyz, types, _ = si.structure(lattice, L, boxes, sp, 0.0, seed=3, images=False, shuffle=False)
    half = si.site_half_units(lattice, L)
    rng = np.random.default_rng(7)
    x = rng.choice([-1.0, 1.0], 200000) * 10.0 ** rng.uniform(17, 20, 200000)
    u = residual(x, L[0], box)
    x, u = x[(u < -1) | (u > m + 1)], u[(u < -1) | (u > m + 1)]
    left = np.arange(N)
    moved = 0
    for xi, r in zip(x[:400], np.rint(u[:400]).astype(np.int64)):
        at = left[half[left, 0] == r % m]
        if len(at):
            xyz[at[0], 0] = xi
            left = left[left != at[0]]
            moved += 1
    assert moved >= 20
    buf = torch.full((3 * N,), -7, dtype=torch.int32, device="cuda")
    out = torch.full((3 * N,), -7, dtype=torch.int8, device="cuda")
    pb.pyhea_map_sites(lattice, L, M, 1, boxes, 0.5, torch.from_numpy(xyz).cuda(), torch.from_numpy(types).cuda(),
                       out[N:2 * N], buf[N:2 * N])
    owner, got = buf.cpu().numpy(), out.cpu().numpy()
    np.testing.assert_array_equal(owner[N:2 * N], np.arange(N))
    np.testing.assert_array_equal(got[N:2 * N], sp)
    for a in (owner, got):
        assert (a[:N] == -7).all() and (a[2 * N:] == -7).all()
