"""Per-cell tags (GPU): with the fused halo and batched launches (3D: every cell
tested once by its own patch, read by its neighbours) equal, byte for byte, to
the other paths (every halo filled beforehand; one launch per patch), which test
each leaf's dilated box by itself, and the requests too.  Walls, mixed and
periodic sides, coarse/fine regions, patch edges that are not whole tiles, every
dilation."""
import numpy as np
import pytest

from oracle.solver import OracleAMR
from paper_2508_05020_amd import workloads as W
from tests import _harness as H

pytestmark = pytest.mark.gpu

LAYOUTS = [(1, 96, [24, 16]), (1, 1920, [24, 16]), (2, 96, [24, 16, 16]), (2, 160, [40, 40]), (3, 24, [12, 8]), (3, 32, [16, 8, 8]),
           (3, 40, [20, 20])]
SIDES = {"walls": [False] * 3, "mixed": [True, False, True], "periodic": [True] * 3}


@pytest.mark.parametrize("sides", SIDES)
@pytest.mark.parametrize("d,base,patches", LAYOUTS)
def test_cell_tags_equal_every_path(d, base, patches, sides):
    import paper_2508_05020_amd.amr as A
    cfg = W.AMRConfig(name="tags", dim=d, base_cells=base, patch_cells=patches, periodic=SIDES[sides][:d],
                      max_patches=2048)
    o = OracleAMR(cfg)
    rng = np.random.default_rng(11)

    def gen(pts):
        # sparse single cells far over the threshold, also at patch and domain edges
        s = 1.0 + 0.5 * (rng.random(pts[0].shape) < 0.02)
        return s, [0.1 * s for _ in pts], 1.0 + 0.2 * (rng.random(s.shape) < 0.01)
    for k in o.forest.keys():
        o.set_initial(k, gen)
    hs = [A.Hierarchy(cfg), A.Hierarchy(cfg), A.Hierarchy(cfg, exec_mode=A.EXEC_PER_PATCH)]
    hs[1].set_fused_halo(False)
    pick = np.random.default_rng(2)
    none = np.zeros(cfg.max_patches, np.uint8)
    for h in hs:
        H.mirror(o, h)
    for _ in range(cfg.max_levels - 1):
        f = none.copy()
        for t in hs[0].patch_table():
            if t["nchildren"] == 0 and t["level"] + 1 < cfg.max_levels:
                f[t["pid"]] = pick.random() < 0.3
        for h in hs:
            h.regrid(f, none)
    leaves = [t for t in hs[0].patch_table() if t["nchildren"] == 0]
    tags = 0
    for b in range(4):
        got = []
        for h in hs:
            h.set_tag_buffer(b)
            r, c, cells = h.tag(0, cell_tags=True)
            flat = cells.cpu().numpy()
            boxes = []
            for t in leaves:
                n, off = patches[t["level"]] + 8, h.offset(t["pid"]) // h.nvar
                boxes.append(H.interior(flat[off:off + n ** d].reshape((1,) + (n,) * d), d).copy())
            got.append((r.cpu().numpy(), c.cpu().numpy(), boxes))
        for other in got[1:]:
            assert np.array_equal(got[0][0], other[0]) and np.array_equal(got[0][1], other[1]), b
            for t, x, y in zip(leaves, got[0][2], other[2]):
                assert np.array_equal(x, y), (b, t["level"], t["coord"])
        tags += sum(int(x.sum()) for x in got[0][2])
    assert tags > 0 or base == 96 and d == 1     # two cells in a hundred: none in the shortest line
    for h in hs:
        h.close()
