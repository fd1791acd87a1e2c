"""Calls that the caller records into a graph of its own (GPU): replayed after
regrids that shorten the lists, each equals the eager call bit for bit.  Every
launch of a recording reads its list, and the 3D tags their patches per level,
from the directory that regrids rewrite."""
import itertools

import numpy as np
import pytest

from tests import _harness as H

pytestmark = pytest.mark.gpu


def lengths(table, cfg):
    """Entries of the work lists of a mesh, from its patch table."""
    d, nlev = cfg.dim, cfg.max_levels
    at = {(t["level"], t["coord"][:d]): t for t in table}
    offs = [o for o in itertools.product((-1, 0, 1), repeat=d) if any(o)]
    np_ = [(cfg.base_cells << l) // cfg.patch_cells[l] for l in range(nlev)]

    def shifted(t, off, clamp):
        q = []
        for c, o, n, per in zip(t["coord"], off, [np_[t["level"]]] * d, cfg.periodic):
            if per:
                q.append((c + o) % n)
            elif 0 <= c + o < n:
                q.append(c + o)
            elif clamp:
                q.append(c)
            else:
                return None
        return at.get((t["level"], tuple(q)))
    leaves = [t for t in table if t["nchildren"] == 0]
    regions = [(t, o) for t in leaves if t["level"] for o in offs if shifted(t, o, True) is None]
    faces = [o for o in offs if sum(map(abs, o)) == 1]
    reflux = [t for t in leaves if any((q := shifted(t, o, False)) and q["nchildren"] for o in faces)]
    parents = {t["parent"] for t in table if t["parent"] >= 0}
    cands = parents - {t["parent"] for t in table if t["nchildren"]}
    n = {"all": len(table), "leaves": len(leaves), "regions": len(regions), "reflux": len(reflux), "cands": len(cands),
         "faces": sum(o in faces for _, o in regions)}
    for l in range(nlev):
        n["leaves", l] = sum(t["level"] == l for t in leaves)
        n["inner", l] = sum(t["level"] == l for t in table) - n["leaves", l]
    n["tiles"] = sum(n["leaves", l] * cfg.patch_cells[l] ** d for l in range(nlev))
    n["boxes"] = sum((n["leaves", l] + n["inner", l]) * cfg.patch_cells[l] ** d for l in range(nlev))
    return n


def calls(h, out):
    """One of each recordable call, into buffers that the caller holds."""
    h.fill_ghosts(0)
    h.velocity_gradient(0, out["gradient"])
    h.rhs(0, out["rhs"])
    h.compute_dt(0, out["dt"])
    out["tags"] = h.tag(0, cell_tags=True)


def buffers(h):
    import torch
    return {"gradient": h.velocity_gradient(0), "rhs": h.new_state_like(),
            "dt": torch.zeros(1, dtype=torch.float64, device="cuda"),
            "step": torch.zeros(1, dtype=torch.float64, device="cuda")}


def boxes(h, flat, table, nvar):
    """Per patch its box of every variable of a flat buffer."""
    host, d, out = flat.detach().cpu().numpy(), h.cfg.dim, {}
    for t in table:
        m = (h.cfg.patch_cells[t["level"]] + 8) ** d
        off = h.offset(t["pid"]) * nvar // h.nvar
        out[t["level"], t["coord"]] = host[off:off + nvar * m].reshape((nvar,) + (h.cfg.patch_cells[t["level"]] + 8,) * d)
    return out


def upload(o, h, table, seed):
    """States of the mesh of `table`, ghosts NaN, the same for the same seed."""
    rng = np.random.default_rng(seed)
    d = o.cfg.dim
    for b in range(3):
        state = {}
        for t in table:
            n = o.cfg.patch_cells[t["level"]]
            u = np.full((d + 2,) + (n + 8,) * d, np.nan)
            inner = H.interior(u, d)
            inner[0] = 1.0 + 0.3 * (rng.random(inner[0].shape) < 0.05) + 0.01 * rng.random(inner[0].shape)
            inner[1:-1] = 0.2 * rng.uniform(-1, 1, inner[1:-1].shape)
            inner[-1] = 2.5 + 0.1 * rng.random(inner[-1].shape)
            state[t["pid"]] = u
        h.set_state(b, state)


def coarsen(h, above):
    """Coarsens every patch of level `above` or finer."""
    none = np.zeros(h.cfg.max_patches, np.uint8)
    for _ in range(h.cfg.max_levels):
        f = none.copy()
        f[[t["pid"] for t in h.patch_table() if t["nchildren"] and t["level"] >= above]] = 1
        h.regrid(none, f)


@pytest.mark.parametrize("fused", [True, False])
@pytest.mark.parametrize("name", ["1d", "2d", "2d-wall", "3d", "3d-uneven"])
def test_replays_follow_regrids(name, fused):
    import torch
    import paper_2508_05020_amd.amr as A
    o, _ = H.oracle_for(name)
    cfg, d = o.cfg, o.cfg.dim
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        hg, he = A.Hierarchy(cfg), A.Hierarchy(cfg)
        outs = []
        for h in (hg, he):
            h.set_fused_halo(fused)
            H.mirror(o, h)
            outs.append(buffers(h))
            calls(h, outs[-1])                    # first launches outside the recording
            h.step(outs[-1]["step"])
        table = hg.patch_table()
        first = lengths(table, cfg)
        for h in (hg, he):
            upload(o, h, table, 0)                # the recorded step forms its own rate
        side.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=side):
            calls(hg, outs[0])
        g2 = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g2, stream=side):
            hg.step(outs[0]["step"])
        compared = 0
        for k in range(cfg.max_levels + 2):
            if 0 < k <= cfg.max_levels:           # one level less each time, then the first mesh again
                for h in (hg, he):
                    coarsen(h, max(cfg.max_levels - 1 - k, 0))
            elif k:
                for level in range(cfg.max_levels - 1):
                    for h in (hg, he):
                        f = np.zeros(cfg.max_patches, np.uint8)
                        at = {(t["level"], t["coord"]): t["pid"] for t in h.patch_table()}
                        f[[at[t["level"], t["coord"]] for t in table if t["level"] == level and t["nchildren"]]] = 1
                        h.regrid(f, np.zeros_like(f))
            now = hg.patch_table()
            assert now == he.patch_table()
            if any(v > first.get(key, 0) for key, v in lengths(now, cfg).items() if key[0] != "leaves"):
                continue                          # longer than the recording covers
            compared += 1
            for h in (hg, he):
                upload(o, h, now, 10 + k)
            for again in range(2):
                g.replay()
                calls(he, outs[1])
                side.synchronize()
                leaves = [t for t in now if t["nchildren"] == 0]
                sg, se = (boxes(h, h.state_tensor(0), now, h.nvar) for h in (hg, he))
                for key in sg:
                    assert np.array_equal(sg[key], se[key], equal_nan=True), (k, key)
                    assert not np.isnan(sg[key]).any(), (k, key)
                a, b = (boxes(h, out["rhs"], leaves, h.nvar) for h, out in ((hg, outs[0]), (he, outs[1])))
                for key in a:
                    assert np.array_equal(H.interior(a[key], d), H.interior(b[key], d)), (k, "rhs", key)
                plane = hg.state_tensor(0).numel() // hg.nvar
                for v in range(d * d + 1):
                    a, b = (boxes(h, out["gradient"].flatten()[v * plane:(v + 1) * plane], leaves, 1)
                            for h, out in ((hg, outs[0]), (he, outs[1])))
                    for key in a:
                        assert np.array_equal(H.interior(a[key], d), H.interior(b[key], d)), (k, v, key)
                assert outs[0]["dt"].item() == outs[1]["dt"].item()
                for a, b in zip(outs[0]["tags"][:2], outs[1]["tags"][:2]):
                    assert torch.equal(a, b), k
                a, b = (boxes(h, out["tags"][2], leaves, 1) for h, out in ((hg, outs[0]), (he, outs[1])))
                for key in a:
                    assert np.array_equal(H.interior(a[key], d), H.interior(b[key], d)), (k, "cells", key)
                g2.replay()
                he.step(outs[1]["step"])
                side.synchronize()
                assert outs[0]["step"].item() == outs[1]["step"].item()
                sg, se = (boxes(h, h.state_tensor(0), now, h.nvar) for h in (hg, he))
                for key in sg:
                    assert np.array_equal(H.interior(sg[key], d), H.interior(se[key], d)), (k, key)
        assert compared >= 3
        assert hg.fill_error() == 0 and he.fill_error() == 0
        hg.close()
        he.close()


CALLS = {"fill": lambda h, out: h.fill_ghosts(0), "gradient": lambda h, out: h.velocity_gradient(0, out["gradient"]),
         "rhs": lambda h, out: h.rhs(0, out["rhs"]), "dt": lambda h, out: h.compute_dt(0, out["dt"]),
         "tags": lambda h, out: out.update(tags=h.tag(0, cell_tags=True)),
         "flags": lambda h, out: out.update(tags=h.tag(0)), "stage": lambda h, out: h.rk_stage(1, out["step"]),
         "step": lambda h, out: h.step(out["step"])}


def results(h, out, call, table):
    """What a call leaves on a mesh, in table order."""
    d, leaves = h.cfg.dim, [t for t in table if t["nchildren"] == 0]
    if call == "fill":
        return list(boxes(h, h.state_tensor(0), table, h.nvar).values())
    if call in ("stage", "step"):
        return [H.interior(b, d) for b in boxes(h, h.state_tensor(1 if call == "stage" else 0), table, h.nvar).values()]
    if call == "dt":
        return [out["dt"].cpu().numpy()]
    if call in ("tags", "flags"):
        cells = boxes(h, out["tags"][2], leaves, 1) if call == "tags" else {}
        return [t.cpu().numpy() for t in out["tags"][:2]] + [H.interior(b, d) for b in cells.values()]
    if call == "rhs":
        return [H.interior(b, d) for b in boxes(h, out["rhs"], leaves, h.nvar).values()]
    plane = h.state_tensor(0).numel() // h.nvar
    return [H.interior(b, d) for v in range(d * d + 1)
            for b in boxes(h, out["gradient"].flatten()[v * plane:(v + 1) * plane], leaves, 1).values()]


@pytest.mark.parametrize("call", CALLS)
@pytest.mark.parametrize("name", ["1d", "2d", "3d", "3d-uneven"])
def test_longer_lists_are_reported(name, call):
    """Recorded on level 0 alone, where the lists of the coarse/fine faces are
    empty: on finer meshes a replay is the eager call, or sets the error flag."""
    import torch
    import paper_2508_05020_amd.amr as A
    o, _ = H.oracle_for(name)
    cfg = o.cfg
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        hg, he = A.Hierarchy(cfg), A.Hierarchy(cfg)
        outs = [buffers(h) for h in (hg, he)]
        base = hg.patch_table()
        for h, out in zip((hg, he), outs):
            upload(o, h, base, 0)
            out["step"].fill_(1e-5)
            CALLS[call](h, out)
            upload(o, h, base, 0)
        side.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=side):
            CALLS[call](hg, outs[0])
        flags = []
        for mesh in ("base", "one", "full", "base again"):
            for h in (hg, he):
                coarsen(h, 0)
                for level in range(cfg.max_levels - 1):
                    at = {(t["level"], t["coord"]): t["pid"] for t in h.patch_table()}
                    want = [k for k in o.forest.keys() if k[0] == level and not o.forest.is_leaf(k)]
                    f = np.zeros(cfg.max_patches, np.uint8)
                    if mesh == "full":
                        f[[at[k] for k in want]] = 1
                    elif mesh == "one" and level == 0:
                        f[at[want[0]]] = 1
                    h.regrid(f, np.zeros_like(f))
            now = hg.patch_table()
            assert now == he.patch_table()
            for h, out in zip((hg, he), outs):
                upload(o, h, now, 5)
                out["step"].fill_(1e-5)
                assert h.fill_error() == 0
            g.replay()
            CALLS[call](he, outs[1])
            side.synchronize()
            flags.append(hg.fill_error())
            assert he.fill_error() == 0
            same = all(np.array_equal(a, b, equal_nan=a.dtype.kind == "f")
                       for a, b in zip(results(hg, outs[0], call, now), results(he, outs[1], call, now)))
            assert same or flags[-1], mesh
        assert flags[0] == flags[3] == 0 and flags[2] == 1, flags
        hg.close()
        he.close()


@pytest.mark.parametrize("warm", [0, 4])
def test_step_in_graph_mode_is_recorded(warm):
    """With the library's own replay enabled a recorded step holds its launches
    (a launch of the library's graph would leave the recording empty)."""
    import torch
    import paper_2508_05020_amd.amr as A
    o, _ = H.oracle_for("2d")
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        hg, he = A.Hierarchy(o.cfg), A.Hierarchy(o.cfg)
        for h in (hg, he):
            H.mirror(o, h)
            h.set_graph(True)
            for _ in range(warm):
                h.step()
            upload(o, h, h.patch_table(), 1)
        dts = [torch.zeros(1, dtype=torch.float64, device="cuda") for _ in range(2)]
        side.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=side):
            hg.step(dts[0])
        table = hg.patch_table()
        for _ in range(3):
            g.replay()
            he.step(dts[1])
            side.synchronize()
            assert dts[0].item() == dts[1].item() > 0
            a, b = (boxes(h, h.state_tensor(0), table, h.nvar) for h in (hg, he))
            for key in a:
                assert np.array_equal(H.interior(a[key], 2), H.interior(b[key], 2)), key
        hg.close()
        he.close()
