"""Ghost fill and prolongation of rough random states (GPU), bit for bit
against the oracle: patch edges of every residue the index products meet (a
power of two, 12, 24, 20), transmissive and periodic walls, and states whose
limited slopes reach non-positive children in some cells and come near it in
others, so that the fast positivity test, the full one and the dropped slopes
are all taken."""
import numpy as np
import pytest

from oracle import euler
from oracle.solver import OracleAMR
from paper_2508_05020_amd import workloads as W
from tests import _harness as H

MESHES = [(1, 64, [16, 8], False), (1, 40, [8, 16], True), (2, 72, [24, 24], False),
          (2, 48, [16, 32], True), (2, 40, [8, 16], False), (3, 36, [12, 12], False),
          (3, 32, [16, 8], True), (3, 60, [20, 8], True)]


def _oracle(d, base, cells, periodic):
    cfg = W.AMRConfig(name="rough", dim=d, base_cells=base, patch_cells=cells,
                      periodic=[periodic] * d, max_patches=4096)
    o = OracleAMR(cfg)
    rng = np.random.default_rng(5)

    def gen(pts):
        # smooth in half of the domain, rough and near vacuum in the other
        x = pts[0]
        rough = x > 0.5
        rho = np.where(rough, 10.0 ** rng.uniform(-4, 0, x.shape), 1.0 + 0.2 * np.sin(6 * x))
        p = np.where(rough, 10.0 ** rng.uniform(-4, 0, x.shape), 1.0 + 0.2 * np.cos(5 * x))
        return rho, [np.where(rough, rng.uniform(-2, 2, x.shape), 0.1) for _ in pts], p
    for k in o.forest.keys():
        o.set_initial(k, gen)
    first, last = (0, (0,) * d), (0, (cfg.patches_per_dim(0) - 1,) * d)
    o.regrid([first, last], [], gen)
    return o


def _dropped(o):
    """Share of the level-0 cells (periodic neighbours) that drop their slopes,
    and that keep them with the smallest child pressure below a fifth of the
    cell's."""
    d = o.d
    u = o.canvas(0, 0)[0]
    sl = []
    for j in range(d):
        ax = d - j
        a = np.roll(u, -1, ax) - u
        b = u - np.roll(u, 1, ax)
        mag = np.minimum(2 * np.minimum(abs(a), abs(b)), 0.5 * abs(a + b))
        sl.append(np.where(a * b > 0, np.sign(a) * mag, 0.0))
    low = np.full(u.shape[1:], np.inf)
    for s in np.ndindex(*(2,) * d):
        ch = u + sum((0.5 * k - 0.25) * v for k, v in zip(s, sl))
        p = euler.primitives(ch, d, o.grid.gamma)[2]
        low = np.minimum(low, np.where(ch[0] > 0, p, -1.0))
    p0 = euler.primitives(u, d, o.grid.gamma)[2]
    return float(np.mean(low <= 0)), float(np.mean((low > 0) & (low < 0.2 * p0)))


@pytest.mark.parametrize("d,base,cells,periodic", MESHES)
def test_rough_states_reach_every_branch(d, base, cells, periodic):
    bad, near = _dropped(_oracle(d, base, cells, periodic))
    assert 0.0 < bad < 0.9 and near > 0.0, (bad, near)


@pytest.mark.gpu
@pytest.mark.parametrize("d,base,cells,periodic", MESHES)
def test_fill_and_prolong_bitwise(d, base, cells, periodic):
    import paper_2508_05020_amd.amr as A
    o = _oracle(d, base, cells, periodic)
    h = A.Hierarchy(o.cfg)
    pid_of, _ = H.mirror(o, h, bufs=(0,))
    h.fill_ghosts(0)
    assert h.fill_error() == 0
    o.fill_ghosts(0)
    got = H.download(h, 0, pid_of)
    for k in o.forest.keys():
        assert np.array_equal(got[k], o.U[0][k]), k
    # a patch refined now: its children are prolonged
    pick = next(k for k in reversed(sorted(o.forest.keys())) if k[0] == 0 and o.forest.is_leaf(k))
    rq = np.zeros(o.cfg.max_patches, np.uint8)
    rq[pid_of[pick]] = 1
    h.regrid(rq, np.zeros_like(rq))
    o.regrid([pick], [])
    pid_of = {(t["level"], t["coord"]): t["pid"] for t in h.patch_table()}
    got = H.download(h, 0, pid_of)
    for k in o.forest.children[pick]:
        assert np.array_equal(H.interior(got[k], d), H.interior(o.U[0][k], d)), k
    h.close()
