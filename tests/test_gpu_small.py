"""Small boxes (at most 3,072 atoms): one work-group per box bins them and reduces the previous step.  The same
bits as the separate kernels, which md_step_timed launches for every box."""
import numpy as np
import pytest

from pe_melt import make_melt

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("chains,precision,kernel,integrator,com,graph", [
    (128, "mixed", 2, "verlet", False, True),       # 2,048 atoms: two per thread
    (129, "fp64", 2, "leapfrog", True, False),      # three per thread
    (129, "mixed", 6, "verlet", True, True),
    (192, "fp64", 1, "verlet", True, True),         # 3,072 atoms: the largest
    (192, "mixed", 1, "leapfrog", False, True),
    (193, "mixed", 2, "verlet", False, False),      # past it: the separate kernels on both sides
])
def test_same_bits_as_the_separate_kernels(ff, chains, precision, kernel, integrator, com, graph):
    """Runs of 1, 12 and 20 steps (one step, one graph of several steps and singles, two of them)."""
    from paper_1001_3764_amd.md import MDSystem
    m = make_melt(chains, chain_len=16, density=0.80, T=450.0, seed_melt=41, seed_vel=42, jitter=0.05)
    kw = dict(chain_len=16, precision=precision, cell_div=1 if kernel == 1 else 2, lj_kernel=kernel,
              integrator=integrator, remove_com=com)
    args = (ff, [m.n_chains], m.box[None, :], [330.0], m.pos, m.vel + np.array([[1e-4], [0.0], [-2e-4]]), m.types)
    print("N=%d %s" % (m.n_atoms, kw), flush=True)
    a, b = MDSystem(*args, use_graph=graph, **kw), MDSystem(*args, use_graph=False, **kw)
    for n in (1, 12, 20):
        a.step(n)
        b.step_timed(n)
        for x, y in zip(a.state(), b.state()):
            assert np.array_equal(x, y)
        for x, y in zip(a.bins(), b.bins()):
            assert np.array_equal(x, y)
        assert a.energies() == b.energies()
        assert np.array_equal(a.forces(), b.forces())
    a.rebuild_bins()
    a.compute_forces()
    assert np.array_equal(a.forces(), b.forces())
    a.close()
    b.close()


def test_batch_of_small_boxes(ff):
    """Three small boxes in one context, each equal to the box alone, bit for bit."""
    from paper_1001_3764_amd.md import MDSystem
    melts = [make_melt(c, chain_len=16, density=0.80, T=400.0, seed_melt=60 + c, seed_vel=3, jitter=0.05)
             for c in (90, 192, 131)]
    cat = [np.concatenate(a, axis=-1) for a in zip(*[(m.pos, m.vel, m.types) for m in melts])]
    kw = dict(chain_len=16, precision="mixed", cell_div=1, lj_kernel=1)
    s = MDSystem(ff, [m.n_chains for m in melts], np.stack([m.box for m in melts]), [300.0, 0.0, 420.0], *cat,
                 use_graph=True, **kw)
    s.step(11)
    p, v = s.state()
    e = s.energies()
    s.close()
    at = 0
    for b, m in enumerate(melts):
        a = MDSystem(ff, [m.n_chains], m.box[None, :], [[300.0, 0.0, 420.0][b]], m.pos, m.vel, m.types, **kw)
        a.step(11)
        pa, va = a.state()
        assert np.array_equal(pa, p[:, at:at + m.n_atoms]) and np.array_equal(va, v[:, at:at + m.n_atoms])
        assert a.energies()[0] == e[b]
        a.close()
        at += m.n_atoms


@pytest.mark.parametrize("precision,kernel", [("mixed", 2), ("fp64", 1)])
@pytest.mark.parametrize("boxes,chains", [(512, 8), (513, 8), (513, 32)])
def test_many_boxes(ff, boxes, chains, precision, kernel):
    """Either side of the line for batches (513 boxes of 128 atoms take the separate kernels, of 512 atoms not)."""
    from paper_1001_3764_amd.md import MDSystem
    m = make_melt(chains, chain_len=16, density=0.09 * chains / 8, T=400.0, seed_melt=81, seed_vel=82, jitter=0.05)
    vel = np.tile(m.vel, (1, boxes)) * np.repeat(1.0 + 0.1 * np.cos(np.arange(boxes)), m.n_atoms)
    args = (ff, [m.n_chains] * boxes, np.tile(m.box, (boxes, 1)), [330.0] * boxes, np.tile(m.pos, (1, boxes)), vel,
            np.tile(m.types, boxes))
    kw = dict(chain_len=16, precision=precision, cell_div=1, lj_kernel=kernel)
    print("%d boxes of %d atoms %s" % (boxes, m.n_atoms, kw), flush=True)
    a, b = MDSystem(*args, use_graph=True, **kw), MDSystem(*args, use_graph=False, **kw)
    a.step(11)
    b.step_timed(11)
    for x, y in zip(a.state(), b.state()):
        assert np.array_equal(x, y)
    assert a.energies() == b.energies()
    a.close()
    b.close()


@pytest.mark.parametrize("precision,kernel", [("mixed", 1), ("fp64", 2)])
@pytest.mark.parametrize("edge", [123.0, 131.5])
def test_sparse_grids(ff, edge, precision, kernel):
    """Either side of the LDS line: 3,000 atoms in 23^3 cells (73 kB of LDS) and in 25^3 (the separate kernels)."""
    from paper_1001_3764_amd.md import MDSystem
    m = make_melt(250, chain_len=12, density=0.045, T=400.0, seed_melt=91, seed_vel=92, jitter=0.05)
    p = m.pos.reshape(3, -1, m.chain_len)
    d = np.diff(p, axis=2)
    d -= m.box[:, None, None] * np.round(d / m.box[:, None, None])
    p = np.concatenate([p[:, :, :1], p[:, :, :1] + np.cumsum(d, axis=2)], axis=2).reshape(3, -1)
    box = np.full(3, edge)
    assert (box > m.box).all()
    args = (ff, [m.n_chains], box[None, :], [330.0], np.ascontiguousarray(np.mod(p, box[:, None])), m.vel, m.types)
    kw = dict(chain_len=12, precision=precision, cell_div=2, lj_kernel=kernel)
    print("N=%d edge %.1f %s" % (m.n_atoms, edge, kw), flush=True)
    a, b = MDSystem(*args, use_graph=True, **kw), MDSystem(*args, use_graph=False, **kw)
    for n in (3, 9):
        a.step(n)
        b.step_timed(n)
        for x, y in zip(a.state() + a.bins(), b.state() + b.bins()):
            assert np.array_equal(x, y)
        assert a.energies() == b.energies()
    a.close()
    b.close()
