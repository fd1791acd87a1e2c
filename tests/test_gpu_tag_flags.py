"""3D tag flags without per-cell output (each cell tested once, masks shared
between neighbours) against the per-patch boxes of the cell-tag path and the
oracle (GPU): exact, for every dilation, on meshes with coarse/fine regions,
transmissive walls, ragged patch edges (partial 8^3 tiles) and magnitudes
outside the range of the reciprocal form."""
import numpy as np
import pytest

from oracle.solver import OracleAMR
from paper_2508_05020_amd import workloads as W
from tests import _harness as H

pytestmark = pytest.mark.gpu

MESHES = ["3d", "3d-uneven", "3d-c5", "ragged", "walls", "scaled", "ragged-sparse", "walls-sparse"]


def _oracle(name):
    if name.startswith("3d"):
        return H.oracle_for(name)[0]
    cells, base, periodic = {"ragged": ([12, 12], 36, [True] * 3), "walls": ([20, 8], 40, [False, True, False]),
                             "scaled": ([8, 4], 32, [True] * 3)}[name.split("-")[0]]
    cfg = W.AMRConfig(name=name, dim=3, base_cells=base, patch_cells=cells, periodic=periodic, max_patches=4096)
    o = OracleAMR(cfg)
    rng = np.random.default_rng(3)

    def gen(pts):
        # steps of about the tag threshold, so that tags are sparse and decided
        # by the last digits in some cells
        s = 1.0 + 0.04 * (np.sin(40 * pts[0] + 3 * pts[1]) > 0.6) * (pts[2] > 0.5)
        if name.endswith("sparse"):   # one small block: few patches, the dilation decides which
            s = 1.0 + 0.2 * (abs(pts[0] - 0.36) < 0.04) * (abs(pts[1] - 0.6) < 0.05) * (abs(pts[2] - 0.3) < 0.04)
        rho = s * (1 + 1e-3 * rng.uniform(-1, 1, s.shape))
        return rho, [rng.uniform(-0.3, 0.3, s.shape) for _ in pts], 1.0 + 0.3 * (s - 1)
    for k in o.forest.keys():
        o.set_initial(k, gen)
    o.regrid([(0, (0, 0, 0)), (0, (cfg.patches_per_dim(0) - 1,) * 3)], [], gen)
    if name == "scaled":
        for i, k in enumerate(o.forest.keys()):
            o.U[0][k] *= 2.0 ** [0, -320, 320, -400][i % 4]
    return o


@pytest.mark.parametrize("name", MESHES)
def test_flags_equal_cell_tag_path(name):
    import paper_2508_05020_amd.amr as A
    o = _oracle(name)
    h = A.Hierarchy(o.cfg)
    pid_of, key_of = H.mirror(o, h, bufs=(0,))
    seen = set()
    for b in range(4):
        h.set_tag_buffer(b)
        r1, c1, _ = h.tag(0)
        r2, c2, cells = h.tag(0, cell_tags=True)
        assert np.array_equal(r1.cpu().numpy(), r2.cpu().numpy()), b
        assert np.array_equal(c1.cpu().numpy(), c2.cpu().numpy()), b
        assert h.judge() == int(r1.cpu().numpy().sum())
        seen.add((int(r1.sum()), int(c1.sum())))
    assert len(seen) > 1 or not name.endswith("sparse"), seen     # the dilation matters
    if name != "scaled":
        h.set_tag_buffer(o.cfg.tag_buffer)
        r1, c1, _ = h.tag(0)
        o.fill_ghosts(0, o.tag_keys())
        oref, ocoa = o.requests(o.tag(0)[0])
        assert {key_of[p] for p in np.nonzero(r1.cpu().numpy())[0]} == set(oref)
        assert {key_of[p] for p in np.nonzero(c1.cpu().numpy())[0]} == set(ocoa)
    h.close()
