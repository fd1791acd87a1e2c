"""The stage kernel's work items (tile, neighbours, parent cell; GPU): with
halos read from the neighbours the items name, three steps with refinement and
coarsening between them equal, bit for bit, the same steps with every halo
copied into ghost layers by the fill kernel beforehand (which works from the
patch tables).  Walls, mixed and periodic sides, ratios 1 to 4, every admissible
tile variant, eager and recorded steps, one launch per item."""
import numpy as np
import pytest

from oracle.solver import OracleAMR
from paper_2508_05020_amd import workloads as W
from tests import _harness as H

LAYOUTS = [(1, 64, [16, 16]), (1, 32, [8, 8, 8]), (2, 64, [16, 16, 16]), (2, 64, [32, 16]), (2, 32, [8, 16]),
           (3, 32, [8, 8]), (3, 32, [16, 8]), (3, 16, [4, 8])]
SIDES = {"walls": [False] * 3, "mixed": [True, False, True], "periodic": [True] * 3}


def _config(d, base, patches, sides):
    return W.AMRConfig(name=f"items{d}", dim=d, base_cells=base, patch_cells=patches, tag_buffer=2,
                       periodic=SIDES[sides][:d], max_patches=1024)


def _smooth(o, seed):
    rng = np.random.default_rng(seed)
    k = rng.uniform(0.5, 1.5, (3, o.cfg.dim)) * 2 * np.pi

    def gen(pts):
        f = [np.sin(sum(k[i, j] * pts[j] for j in range(o.cfg.dim))) for i in range(3)]
        return 1.0 + 0.4 * f[0], [0.3 * f[1] for _ in pts], 1.0 + 0.4 * f[2]
    for key in o.forest.keys():
        o.set_initial(key, gen)


def _flags(h, rng, refine):
    """Random requests on what is there: leaves to refine, or parents to coarsen."""
    f = np.zeros(h.cfg.max_patches, np.uint8)
    for t in h.patch_table():
        if refine == (t["nchildren"] == 0) and t["level"] + 1 < h.cfg.max_levels:
            f[t["pid"]] = rng.random() < 0.25
    return f


def _run(A, o, fused, variant, graph=False, mode=None):
    h = A.Hierarchy(o.cfg, **({} if mode is None else {"exec_mode": mode}))
    H.mirror(o, h)
    try:
        h.set_tile_variant(variant)
    except A.AMRError:
        h.close()
        return None
    h.set_fused_halo(fused)
    if graph:
        h.set_graph(True)
    rng = np.random.default_rng(5)
    none = np.zeros(h.cfg.max_patches, np.uint8)
    h.regrid(_flags(h, rng, True), none)
    for refine in (True, False, None):
        h.step()
        if refine is not None:
            f = _flags(h, rng, refine)
            h.regrid(f if refine else none, none if refine else f)
    leaves = {(t["level"], t["coord"]): t["pid"] for t in h.patch_table() if t["nchildren"] == 0}
    got = H.download(h, 0, leaves)
    assert h.fill_error() == 0
    h.close()
    return got


@pytest.mark.gpu
@pytest.mark.parametrize("sides", SIDES)
@pytest.mark.parametrize("d,base,patches", LAYOUTS)
def test_items_equal_filled_ghosts(d, base, patches, sides):
    import paper_2508_05020_amd.amr as A
    o = OracleAMR(_config(d, base, patches, sides))
    _smooth(o, 9)
    done = 0
    for v in range(11):
        ref = _run(A, o, False, v)
        if ref is None:
            continue
        runs = [dict(), dict(graph=True)] + ([dict(mode=A.EXEC_PER_PATCH)] if done == 0 else [])
        for kw in runs:
            got = _run(A, o, True, v, **kw)
            assert set(got) == set(ref)
            for k in ref:
                assert np.array_equal(H.interior(got[k], d), H.interior(ref[k], d)), (v, kw, k)
        done += 1
    assert done >= 1
