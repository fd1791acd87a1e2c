"""3D tags by the shared flags (each cell tested once, quotients by one reciprocal)
against the routes that test every leaf's dilated box with divisions (GPU): all
halos filled beforehand, and one launch per patch.  Requests exact, with and
without per-cell output, and the cells' tags, for every dilation, on meshes with
coarse/fine regions, walls, ragged patch edges and magnitudes outside the
reciprocal form's range."""
import numpy as np
import pytest

from tests import _harness as H
from tests.test_gpu_tag_flags import MESHES, _oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name", MESHES)
def test_shared_flags_equal_the_boxes(name):
    import paper_2508_05020_amd.amr as A
    o = _oracle(name)
    shared, filled = A.Hierarchy(o.cfg), A.Hierarchy(o.cfg)
    filled.set_fused_halo(False)
    per_patch = A.Hierarchy(o.cfg, exec_mode=A.EXEC_PER_PATCH)
    hs = (shared, filled, per_patch)
    for h in hs:
        H.mirror(o, h, bufs=(0,))
    leaves = [t for t in shared.patch_table() if t["nchildren"] == 0]
    tagged = untagged = 0
    for b in range(4):
        got, boxes = [], []
        for h in hs:
            h.set_tag_buffer(b)
            got.append([t.cpu().numpy() for t in h.tag(0)[:2]])
            r, c, cells = (t.cpu().numpy() for t in h.tag(0, cell_tags=True))
            got.append([r, c])
            box = {}
            for t in leaves:
                n, off = o.cfg.patch_cells[t["level"]] + 8, h.offset(t["pid"]) // h.nvar
                box[t["level"], t["coord"]] = H.interior(cells[off:off + n ** 3].reshape(1, n, n, n), 3)
            boxes.append(box)
        for r, c in got[1:]:
            assert np.array_equal(got[0][0], r) and np.array_equal(got[0][1], c), b
        for key, x in boxes[0].items():
            assert all(np.array_equal(x, other[key]) for other in boxes[1:]), (b, key)
            tagged, untagged = tagged + int(x.sum()), untagged + int((x == 0).sum())
        assert len({h.judge() for h in hs}) == 1
    assert tagged > 0 and untagged > 0
    for h in hs:
        assert h.fill_error() == 0
        h.close()
