"""Steps recorded by the caller into a graph of its own (GPU): replays equal
eager launches bit for bit, also after regrids that make the lists shorter
(the recorded launches read lists and counts from the directory that the
regrids rewrite)."""
import numpy as np
import pytest

from tests import _harness as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name", ["1d", "2d", "3d"])
def test_caller_graph_replays_across_regrids(name):
    import torch
    import paper_2508_05020_amd.amr as A
    o, _ = H.oracle_for(name)
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        hg, he = A.Hierarchy(o.cfg), A.Hierarchy(o.cfg)
        pid, _ = H.mirror(o, hg)
        H.mirror(o, he)
        dt = torch.full((1,), 1e-4, dtype=torch.float64, device="cuda")
        for h in (hg, he):                       # first launches outside the recording
            for stage in (1, 2, 3):
                h.rk_stage(stage, dt)
        side.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=side):
            for stage in (1, 2, 3):
                hg.rk_stage(stage, dt)
        none = np.zeros(o.cfg.max_patches, np.uint8)
        for k in range(4):
            g.replay()
            for stage in (1, 2, 3):
                he.rk_stage(stage, dt)
            side.synchronize()
            table = {(t["level"], t["coord"]): t["pid"] for t in hg.patch_table()}
            a, b = H.download(hg, 0, table), H.download(he, 0, table)
            for key in table:
                assert np.array_equal(H.interior(a[key], o.cfg.dim), H.interior(b[key], o.cfg.dim)), (k, key)
            if k == 1:                           # down to level 0: every list shorter
                for _ in range(o.cfg.max_levels):
                    f = none.copy()
                    f[[t["pid"] for t in hg.patch_table() if t["nchildren"]]] = 1
                    assert hg.regrid(none, f) == he.regrid(none, f)
                assert all(t["level"] == 0 for t in hg.patch_table())
        hg.close()
        he.close()
