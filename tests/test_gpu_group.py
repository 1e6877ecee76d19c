"""GPU parity of the group Lennard-Jones kernel (MD_LJ_ATOM, and every FP64 cell-path kernel) where its
branches change: one or several wavefronts per group, both in one batch, candidate lists longer than one
chunk, groups split by their extent."""
import numpy as np
import pytest

import oracle as O
from pe_melt import make_melt

pytestmark = pytest.mark.gpu

TOL = {"mixed": 1e-5, "fp64": 1e-10}   # max force error over the oracle's RMS force (FP32 / FP64 forces)


def norm_err(f, ref):
    return float(np.max(np.sqrt(np.sum((f - ref) ** 2, axis=0))) / np.sqrt(np.mean(np.sum(ref ** 2, axis=0))))


def system(ff, melts, precision, R, kernel, **kw):
    from paper_1001_3764_amd.md import MDSystem
    print("system: N=%s precision=%s R=%d kernel=%d" % ([m.n_atoms for m in melts], precision, R, kernel), flush=True)
    cat = [np.concatenate(a, axis=-1) for a in zip(*[(m.pos, m.vel, m.types) for m in melts])]
    return MDSystem(ff, [m.n_chains for m in melts], np.stack([m.box for m in melts]), [0.0] * len(melts), *cat,
                    chain_len=melts[0].chain_len, precision=precision, cell_div=R, lj_kernel=kernel, **kw)


@pytest.mark.parametrize("precision,kernel", [("mixed", 1), ("fp64", 1), ("fp64", 2)])
@pytest.mark.parametrize("chains,R", [(49, 1), (49, 2), (70, 1), (70, 2), (70, 3)])
def test_either_side_of_the_split(ff, chains, R, precision, kernel):
    """14,700 atoms have at most 2,048 groups (several wavefronts share one), 21,000 more (one each)."""
    if R == 3 and kernel != 1:
        pytest.skip("cell_div = 3 is MD_LJ_ATOM's")
    m = make_melt(chains, density=0.80, T=500.0, seed_melt=310 + chains, seed_vel=311, jitter=0.05)
    s = system(ff, [m], precision, R, kernel)
    fo, eo = O.forces(ff, m.pos, m.types, m.box, 300)
    err = norm_err(s.forces(), fo)
    e = s.energies()[0]
    s.close()
    print("force error %.3e" % err)
    assert err <= TOL[precision]
    assert e["e_lj"] == pytest.approx(eo["e_lj"], rel=2e-6 if precision == "mixed" else 1e-12)


@pytest.mark.parametrize("precision", ["mixed", "fp64"])
def test_batch_of_both_kinds(ff, precision):
    """A box on each side of the split in one context: each equals the box alone, bit for bit."""
    melts = [make_melt(c, density=0.80, T=400.0, seed_melt=500 + c, seed_vel=501, jitter=0.05) for c in (9, 70, 12)]
    s = system(ff, melts, precision, 2, 1)
    s.step(3)
    p, v = s.state()
    e = s.energies()
    s.close()
    at = 0
    for b, m in enumerate(melts):
        a = system(ff, [m], precision, 2, 1)
        a.step(3)
        pa, va = a.state()
        ea = a.energies()[0]
        a.close()
        assert np.array_equal(pa, p[:, at:at + m.n_atoms]) and np.array_equal(va, v[:, at:at + m.n_atoms])
        assert ea["e_lj"] == e[b]["e_lj"] and ea["virial"] == e[b]["virial"]
        at += m.n_atoms


@pytest.mark.parametrize("precision", ["mixed", "fp64"])
@pytest.mark.parametrize("R,chains", [(1, 24), (2, 24), (2, 75)])
def test_more_than_a_chunk_of_candidates(ff, R, chains, precision):
    """A melt squeezed to 0.55 of its box edge (6 times the density): a group's rows hold more than the
    4,096 candidates whose run starts are marked at a time (also with one wavefront per group)."""
    m = make_melt(chains, density=0.80, T=500.0, seed_melt=77, seed_vel=78, jitter=0.05)
    import dataclasses
    m = dataclasses.replace(m, pos=np.ascontiguousarray(m.pos * 0.55), box=m.box * 0.55)
    s = system(ff, [m], precision, R, 1)
    fo, _ = O.forces(ff, m.pos, m.types, m.box, 300)
    err = norm_err(s.forces(), fo)
    s.close()
    print("force error %.3e" % err)
    assert err <= TOL[precision]


@pytest.mark.parametrize("precision", ["mixed", "fp64"])
@pytest.mark.parametrize("scale", [1.0, 3.0])
def test_sparse_rows(ff, precision, scale):
    """Short chains spread thinly (scale stretches the box, to 209 A along x): the homes of a group lie
    further apart than one group may extend, past the 128 A the fixed-point offsets tell apart."""
    m = make_melt(12, chain_len=24, density=0.02, T=500.0, seed_melt=9, seed_vel=10, jitter=0.05)
    box = m.box * np.array([scale, 1.0, 1.0])
    pos = m.pos.copy()
    # whole chains are moved: x of the first site stretched, the chain carried along
    x = pos[0].reshape(12, 24)
    d = np.diff(x, axis=1)
    d -= m.box[0] * np.round(d / m.box[0])
    x = x[:, :1] * scale + np.concatenate([np.zeros((12, 1)), np.cumsum(d, axis=1)], axis=1)
    pos[0] = np.mod(x.reshape(-1), box[0])
    import dataclasses
    m = dataclasses.replace(m, pos=np.ascontiguousarray(pos), box=box)
    s = system(ff, [m], precision, 2, 1)
    fo, _ = O.forces(ff, m.pos, m.types, m.box, 24)
    flj, _ = O.lj_brute(ff, m.pos, m.types, m.box, 24)
    err, err_lj = norm_err(s.forces(), fo), norm_err(s.forces(lj_only=True), flj)
    s.close()
    print("force error %.3e, LJ %.3e" % (err, err_lj))
    assert err <= TOL[precision] and err_lj <= TOL[precision]


@pytest.mark.parametrize("precision", ["mixed", "fp64"])
@pytest.mark.parametrize("R", [2, 3])
def test_tuned_choice_is_accepted(ff, R, precision):
    """What md_tuning reports for a given cell_div sets up the same context when it is given."""
    m = make_melt(10, density=0.80, T=500.0, seed_melt=1000, seed_vel=1001, jitter=0.05)
    s = system(ff, [m], precision, R, 0)
    r, k, h = s.tuning(homes=True)
    f = s.forces()
    s.close()
    assert r == R
    s = system(ff, [m], precision, r, k, tile_homes=h)
    assert s.tuning(homes=True) == (r, k, h) and np.array_equal(s.forces(), f)
    s.close()


@pytest.mark.parametrize("precision", ["mixed", "fp64"])
@pytest.mark.parametrize("boxes", [4, 5])
def test_batch_on_either_side_of_the_split(ff, boxes, precision):
    """Boxes of 448 groups each: four have fewer than 2,048 together (several wavefronts per group), five more."""
    melts = [make_melt(10, density=0.80, T=400.0, seed_melt=700 + b, seed_vel=701, jitter=0.05) for b in range(boxes)]
    s = system(ff, melts, precision, 2, 1)
    f, e = s.forces(), s.energies()
    s.step(2)
    p, v = s.state()
    s.close()
    for b, m in enumerate(melts):
        fo, eo = O.forces(ff, m.pos, m.types, m.box, 300)
        assert norm_err(f[:, 3000 * b:3000 * (b + 1)], fo) <= TOL[precision]
        assert e[b]["e_lj"] == pytest.approx(eo["e_lj"], rel=2e-6 if precision == "mixed" else 1e-12)
    s = system(ff, melts, precision, 2, 1)
    s.step(2)
    assert all(np.array_equal(x, y) for x, y in zip(s.state(), (p, v)))   # the same every run
    s.close()


@pytest.mark.parametrize("precision", ["mixed", "fp64"])
@pytest.mark.parametrize("R,scale", [(1, 2.0), (2, 2.0), (1, 6.0), (2, 6.0)])
def test_droplet(ff, R, scale, precision):
    """A melt of whole chains in the middle of a larger box: few groups in thin rows (groups of two homes, on more
    blocks), and with 2,500 rows in a nearly empty box (rows gone through eight times)."""
    import dataclasses
    m = make_melt(10, density=0.80, T=500.0, seed_melt=1000, seed_vel=1001, jitter=0.05)
    p = m.pos.reshape(3, -1, m.chain_len)
    d = np.diff(p, axis=2)
    d -= m.box[:, None, None] * np.round(d / m.box[:, None, None])
    flat = np.concatenate([p[:, :, :1], p[:, :, :1] + np.cumsum(d, axis=2)], axis=2).reshape(3, -1)
    box = m.box * scale
    pos = np.mod(flat + 0.5 * (box - m.box)[:, None], box[:, None])
    pos[pos >= box[:, None]] = 0.0
    m = dataclasses.replace(m, pos=np.ascontiguousarray(pos), box=box)
    s = system(ff, [m], precision, R, 1)
    f, flj, e = s.forces(), s.forces(lj_only=True), s.energies()[0]
    s.close()
    fo, eo = O.forces(ff, m.pos, m.types, m.box, 300, R=1)
    lo, _ = O.lj_brute(ff, m.pos, m.types, m.box, 300)
    assert norm_err(f, fo) <= TOL[precision] and norm_err(flj, lo) <= TOL[precision]
    assert e["e_lj"] == pytest.approx(eo["e_lj"], rel=2e-6 if precision == "mixed" else 1e-12)
