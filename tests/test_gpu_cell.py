"""GPU parity of the mixed cell kernels (MD_LJ_CELLTILE, MD_LJ_CELLTILE_NB) where their branches change: rows cut
by the box's edge on the smallest grids, more candidates than are held or marked at a time, cells of more homes
than one pass takes, two LJ types."""
import dataclasses

import numpy as np
import pytest

import oracle as O
from pe_melt import make_melt

pytestmark = pytest.mark.gpu

TOL = 1e-5   # max force error over the oracle's RMS force (FP32 forces)


def check(ff, m, R, kernel, homes):
    from paper_1001_3764_amd.md import MDSystem
    print("N=%d box=%s R=%d kernel=%d homes=%d" % (m.n_atoms, m.box, R, kernel, homes), flush=True)
    s = MDSystem(ff, [m.n_chains], m.box[None, :], [0.0], m.pos, m.vel, m.types, chain_len=m.chain_len,
                 precision="mixed", cell_div=R, lj_kernel=kernel, tile_homes=homes)
    f, e = s.forces(), s.energies()[0]
    s.close()
    fo, eo = O.forces(ff, m.pos, m.types, m.box, m.chain_len, R=R)
    err = float(np.max(np.sqrt(np.sum((f - fo) ** 2, axis=0))) / np.sqrt(np.mean(np.sum(fo ** 2, axis=0))))
    print("force error %.3e" % err)
    assert err <= TOL
    assert e["e_lj"] == pytest.approx(eo["e_lj"], rel=2e-6)


@pytest.mark.parametrize("kernel,homes", [(2, 4), (2, 8), (3, 8), (2, 16)])
@pytest.mark.parametrize("R,edge,chains", [(1, 33.0, 50), (2, 27.0, 28), (2, 33.0, 50)])
def test_smallest_grids(ff, R, edge, chains, kernel, homes):
    """2R + 1 cells along every edge (every row crosses it), and one more."""
    m = make_melt(chains, chain_len=24, density=0.80, T=500.0, seed_melt=60 + chains, seed_vel=61, jitter=0.05)
    m = dataclasses.replace(m, pos=np.ascontiguousarray(m.pos * (edge / m.box)[:, None]), box=np.full(3, edge))
    check(ff, m, R, kernel, homes)


@pytest.mark.parametrize("kernel,homes", [(2, 8), (3, 16)])
@pytest.mark.parametrize("R", [1, 2])
def test_crowded_cells(ff, R, kernel, homes):
    """A melt squeezed to 0.55 of its box edge: stencils of more than 4,096 candidates (R = 1), cells of more
    than 16 atoms, several fills of the candidate list."""
    m = make_melt(24, density=0.80, T=500.0, seed_melt=77, seed_vel=78, jitter=0.05)
    check(ff, dataclasses.replace(m, pos=np.ascontiguousarray(m.pos * 0.55), box=m.box * 0.55), R, kernel, homes)


@pytest.mark.parametrize("R,homes", [(1, 8), (2, 4), (2, 8), (2, 16)])
def test_two_types(ff, R, homes):
    ff = dict(ff)
    ff.update(sigma=(3.47, 3.70), epsilon=(0.0951, 0.1200))
    check(ff, make_melt(10, density=0.80, T=500.0, seed_melt=5, seed_vel=6, jitter=0.05), R, 2, homes)
