"""Host side of the library's calls, without a GPU: tests/fake_hip.c stands in
for the HIP runtime in a process of its own."""
import json
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CC = shutil.which("gcc") or shutil.which("cc")

HEAD = """
import ctypes as C, itertools, json, sys
import numpy as np
fake = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)      # ahead of the HIP runtime
for f in (fake.fake_rewritten, fake.fake_launches, fake.fake_blocks):
    f.restype = C.c_long
sys.path.insert(0, sys.argv[2])
from paper_2508_05020_amd import amr as A, workloads as W

class Host:
    def __init__(self, cfg, mode=A.EXEC_BATCHED):
        self.cfg, self.c, self.h = cfg, A.make_config(cfg, mode), C.c_void_p()
        self.ok(A._lib.amr_create_hierarchy(C.byref(self.c), None, None, C.byref(self.h)))
    def ok(self, st):
        assert st == 0, A._lib.amr_last_error(self.h)
    def call(self, name, *args):
        before = fake.fake_launches()
        self.ok(getattr(A._lib, "amr_" + name)(self.h, *args))
        return fake.fake_launches() - before
    def table(self):
        n = C.c_int()
        rows = (A.PatchInfo * self.cfg.max_patches)()
        self.ok(A._lib.amr_get_patch_table(self.h, rows, self.cfg.max_patches, C.byref(n)))
        return list(rows[:n.value])
    def regrid(self, refine=(), coarsen=()):
        flags = [np.zeros(self.cfg.max_patches, np.uint8) for _ in range(2)]
        for f, pids in zip(flags, (refine, coarsen)):
            f[list(pids)] = 1
        n = C.c_int()
        self.call("regrid", *(f.ctypes.data_as(C.c_void_p) for f in flags), C.byref(n), C.byref(n))
"""


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    if CC is None:
        pytest.skip("no C compiler")
    out = str(tmp_path_factory.mktemp("fake") / "libfake_hip.so")
    subprocess.run([CC, "-O1", "-shared", "-fPIC", os.path.join(ROOT, "tests", "fake_hip.c"), "-o", out], check=True)
    return out


def run(fake, body):
    r = subprocess.run([sys.executable, "-c", HEAD + body, fake, ROOT], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    return json.loads(r.stdout.splitlines()[-1])


@pytest.mark.parametrize("dim,base,patches", [(1, 64, [16, 16]), (2, 64, [16, 16, 16]), (3, 32, [8, 8])])
def test_upload_staging_is_not_rewritten_before_its_copy(fake, dim, base, patches):
    """A regrid's upload may still be reading the pinned staging when the next
    call rebuilds the lists in it: autotuning tried its first variant's lists
    there without waiting."""
    got = run(fake, f"""
cfg = W.AMRConfig(name="up", dim={dim}, base_cells={base}, patch_cells={patches}, periodic=[True] * {dim},
                  max_patches=1024)
h = Host(cfg)
tiles = {{1: (0, 1), 2: (2, 3, 4, 8), 3: (5, 6, 7)}}[{dim}]
best, ms = C.c_int(), C.c_float()
for v in tiles:
    h.call("set_tile_variant", v)
    for _ in range(2):
        leaf = [t.pid for t in h.table() if t.nchildren == 0 and t.level == 0]
        h.regrid(refine=leaf[:2])
        h.regrid(coarsen=[t.pid for t in h.table() if t.nchildren])
    h.regrid(refine=leaf[1:2])
    h.call("autotune", 1, C.byref(best), C.byref(ms))
    h.regrid(refine=leaf[:1])
    h.call("set_tile_variant", tiles[0])
    h.regrid(coarsen=[t.pid for t in h.table() if t.nchildren])
print(json.dumps(fake.fake_rewritten()))
A._lib.amr_destroy_hierarchy(h.h)
""")
    assert got == 0


@pytest.mark.parametrize("dim,base,patches", [(1, 64, [16, 16, 16]), (2, 64, [16, 16, 16]), (3, 32, [8, 8, 8])])
def test_filled_tags_prolong_each_region_once(fake, dim, base, patches):
    """Tags with every halo filled beforehand: the fill of the coarsening
    candidates, which have no prolonged ghosts, repeated that of the leaves."""
    got = run(fake, f"""
cfg = W.AMRConfig(name="tag", dim={dim}, base_cells={base}, patch_cells={patches}, periodic=[True] * {dim},
                  max_patches=2048)
out = []
for mode in (A.EXEC_PER_PATCH, A.EXEC_BATCHED):
    h = Host(cfg, mode)
    h.call("set_fused_halo", 0)
    h.regrid(refine=[h.table()[0].pid])
    h.regrid(refine=[next(t.pid for t in h.table() if t.level == 1)])
    t = h.table()
    inner = set(r.pid for r in t if r.nchildren)
    leaves = len(t) - len(inner)
    cands = len(inner - set(r.parent for r in t if r.pid in inner))
    fill = h.call("fill_ghosts", 0)
    flags = (C.c_uint8 * cfg.max_patches)()
    out.append([len(t), leaves, cands, fill, h.call("tag", 0, flags, flags, None)])
    A._lib.amr_destroy_hierarchy(h.h)
print(json.dumps(out))
""")
    (active, leaves, cands, fill, tag), batched = got
    regions = fill - active
    assert regions > 0 and cands > 0
    # fills of the leaves, their regions and the candidates, a test of each, the requests
    assert tag == 2 * leaves + regions + 2 * cands + 1
    if dim == 3:        # copies and regions of the leaves, copies of the candidates, two tests, the requests
        assert batched[4] == 6
