"""GPU parity at the limits of the force field that the set-up accepts."""
import numpy as np
import pytest

import oracle as O
from pe_melt import make_melt

pytestmark = pytest.mark.gpu

TOL = {"mixed": 1e-5, "fp64": 1e-10}   # max force error over the oracle's RMS force (FP32 / FP64 forces)


def system(ff, m, precision, R, kernel, **kw):
    from paper_1001_3764_amd.md import MDSystem
    print("system: N=%d box=%s precision=%s R=%d kernel=%d" % (m.n_atoms, m.box, precision, R, kernel), flush=True)
    return MDSystem(ff, [m.n_chains], m.box[None, :], [0.0], m.pos, m.vel, m.types, chain_len=m.chain_len,
                    precision=precision, cell_div=R, lj_kernel=kernel, **kw)


def norm_err(f, ref):
    return float(np.max(np.sqrt(np.sum((f - ref) ** 2, axis=0))) / np.sqrt(np.mean(np.sum(ref ** 2, axis=0))))


@pytest.mark.parametrize("precision,R,kernel,skin", [
    ("mixed", 1, 1, 0.0), ("mixed", 2, 1, 0.0), ("mixed", 2, 2, 0.0), ("mixed", 2, 3, 0.0), ("mixed", 2, 6, 0.0),
    ("mixed", 2, 4, 0.8), ("mixed", 2, 5, 0.8), ("fp64", 2, 1, 0.0), ("fp64", 2, 4, 0.8), ("fp64", 2, 5, 0.8)])
def test_no_lennard_jones(ff, precision, R, kernel, skin):
    """epsilon = 0 for both types: the Lennard-Jones force and energies are exactly zero, the rest is the bonded terms."""
    ff = dict(ff, epsilon=(0.0, 0.0))
    m = make_melt(50, chain_len=24, density=0.80, T=500.0, seed_melt=21, seed_vel=22, jitter=0.05)
    s = system(ff, m, precision, R, kernel, **({"nl_skin": skin} if skin else {}))
    f, flj, e = s.forces(), s.forces(lj_only=True), s.energies()[0]
    s.step(3)
    p, v = s.state()
    s.close()
    fo, eo = O.bonded(ff, m.pos, m.box, m.chain_len)
    assert not flj.any() and e["e_lj"] == 0.0 and e["e_lj_shifted"] == 0.0
    assert norm_err(f, fo) <= TOL[precision]
    assert e["virial"] == pytest.approx(eo["virial_bonded"], rel=2e-6 if precision == "mixed" else 1e-12, abs=1e-2)
    assert np.isfinite(p).all() and np.isfinite(v).all()


@pytest.mark.parametrize("precision,R,kernel,skin", [
    ("mixed", 1, 1, 0.0), ("mixed", 2, 1, 0.0), ("mixed", 1, 2, 0.0), ("mixed", 2, 2, 0.0), ("mixed", 2, 3, 0.0),
    ("mixed", 2, 6, 0.0), ("mixed", 2, 4, 0.3), ("mixed", 2, 5, 0.3), ("fp64", 2, 1, 0.0)])
@pytest.mark.parametrize("two_types", [False, True])
def test_cutoff_below_the_close_contacts(ff, two_types, precision, R, kernel, skin):
    """A cutoff below 0.75 sigma, where every pair is a close contact, in a squeezed melt, with pairs so near the
    cutoff that FP32 cannot tell their side (rc is set by the distance of a pair of the configuration)."""
    import dataclasses
    m = make_melt(40, chain_len=24, density=0.80, T=500.0, seed_melt=31, seed_vel=32, jitter=0.05)
    m = dataclasses.replace(m, pos=np.ascontiguousarray(m.pos * 0.7), box=m.box * 0.7)
    from scipy.spatial import cKDTree
    tree = cKDTree(np.mod(m.pos.T, m.box), boxsize=m.box)
    i, j = tree.query_pairs(2.4, output_type="ndarray").T
    far = (i // m.chain_len != j // m.chain_len) | (np.abs(i - j) > 2)
    d = m.pos[:, i] - m.pos[:, j]
    d -= m.box[:, None] * np.round(d / m.box[:, None])
    r = np.sort(np.sqrt(np.sum(d * d, axis=0))[far])
    ff = dict(ff, rc=float(r[-1] * (1.0 + 2e-7)))
    if two_types:
        ff.update(sigma=(3.47, 3.70), epsilon=(0.0951, 0.1200))
    s = system(ff, m, precision, R, kernel, **({"nl_skin": skin} if skin else {}))
    flj, e = s.forces(lj_only=True), s.energies()[0]
    s.close()
    fo, eo = O.lj_brute(ff, m.pos, m.types, m.box, m.chain_len)
    err = norm_err(flj, fo)
    print("rc %.6f, %d pairs, force error %.3e" % (ff["rc"], far.sum(), err))
    assert err <= TOL[precision]
    assert e["e_lj"] == pytest.approx(eo["e_lj"], rel=2e-6 if precision == "mixed" else 1e-12)


@pytest.mark.parametrize("R,kernel", [(1, 1), (2, 1), (2, 2), (3, 1)])
@pytest.mark.parametrize("power", [-33, 12, 18])
def test_other_units_of_length(ff, power, R, kernel):
    """Every length multiplied by a power of two (FP64, whose lengths have no range of their own): the same
    system in another unit, so the forces scale by its inverse."""
    import dataclasses
    u = 2.0 ** power
    m = make_melt(50, chain_len=24, density=0.80, T=500.0, seed_melt=21, seed_vel=22, jitter=0.05)
    fo, eo = O.lj_brute(ff, m.pos, m.types, m.box, m.chain_len)
    ff = dict(ff, sigma=tuple(u * x for x in ff["sigma"]), rc=u * ff["rc"], b0=u * ff["b0"], kb=ff["kb"] / (u * u))
    m = dataclasses.replace(m, pos=u * m.pos, box=u * m.box)
    s = system(ff, m, "fp64", R, kernel)
    flj, e = s.forces(lj_only=True), s.energies()[0]
    s.close()
    err = norm_err(u * flj, fo)
    print("force error %.3e" % err)
    assert err <= TOL["fp64"]
    assert e["e_lj"] == pytest.approx(eo["e_lj"], rel=1e-12)


@pytest.mark.parametrize("R,kernel", [(1, 1), (2, 2), (3, 1)])
@pytest.mark.parametrize("axis", [0, 1, 2])
def test_pairs_across_the_edge_of_a_long_box(ff, axis, R, kernel):
    """FP64, a melt that lies across the edge of a box 1,000 A long.  Each pair's force is the one of the given
    positions to the rounding of differences of at most 64 A: per atom, the error is at most
    sum_j |F_ij| (14 delta / r + 32 ulp), where 14 bounds -d ln F / d ln r away from the force's zero, as computed
    here from F's two terms, and delta = 3 roundings of 2^-48 A (half an ulp below 64 A)."""
    import dataclasses
    m = make_melt(30, chain_len=24, density=0.80, T=500.0, seed_melt=41, seed_vel=42, jitter=0.05)
    p = m.pos.reshape(3, -1, m.chain_len)
    d = np.diff(p, axis=2)
    d -= m.box[:, None, None] * np.round(d / m.box[:, None, None])
    flat = np.concatenate([p[:, :, :1], p[:, :, :1] + np.cumsum(d, axis=2)], axis=2).reshape(3, -1)
    box = np.array([80.0, 80.0, 80.0])   # (whole chains stick out of the original box: no overlaps across the edges)
    box[axis] = 1000.3
    flat[axis] -= 0.5 * m.box[axis]
    pos = np.mod(flat, box[:, None])
    pos[pos >= box[:, None]] = 0.0
    m = dataclasses.replace(m, pos=np.ascontiguousarray(pos), box=box)
    s = system(ff, m, "fp64", R, kernel)
    f = s.forces(lj_only=True)
    s.close()
    from scipy.spatial import cKDTree
    i, j = cKDTree(pos.T, boxsize=box).query_pairs(ff["rc"], output_type="ndarray").T
    k = (i // m.chain_len != j // m.chain_len) | (np.abs(i - j) > ff["excl_depth"])
    i, j = i[k], j[k]
    X = np.longdouble
    d = pos.astype(X)[:, i] - pos.astype(X)[:, j]
    d -= box.astype(X)[:, None] * np.rint(d / box.astype(X)[:, None])
    r2 = np.sum(d * d, axis=0)
    s6 = (X(ff["sigma"][0]) ** 2 / r2) ** 3
    a, b = 48 * X(ff["epsilon"][0]) * s6 * s6 / r2, 24 * X(ff["epsilon"][0]) * s6 / r2
    fo, bound = np.zeros((3, m.n_atoms), X), np.zeros(m.n_atoms, X)
    term = (a + b) * np.sqrt(r2) * (14 * X(3 * 2.0 ** -48) / np.sqrt(r2) + 32 * X(2.0 ** -52))
    for q in range(3):
        np.add.at(fo[q], i, (a - b) * d[q])
        np.add.at(fo[q], j, -(a - b) * d[q])
    np.add.at(bound, i, term)
    np.add.at(bound, j, term)
    err = np.sqrt(np.sum((f - fo) ** 2, axis=0))
    crosses = np.abs(pos[axis][i] - pos[axis][j]) > 500.0
    print("%d of %d pairs across the edge; error over bound %.3f" % (crosses.sum(), i.size, float(np.max(err / bound))))
    assert crosses.sum() > 1000
    assert np.all(err <= bound)
