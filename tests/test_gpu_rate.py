"""The CFL rate (GPU): dt of random states against the definition, cfl / max of
sum_j (|u_j| + c) / h, bit for bit (the largest cell's quotients, root and sums are
the rounded ones), for one to thousands of blocks, values outside the range of
the reciprocal form, and not-a-number."""
import numpy as np
import pytest

from oracle.solver import OracleAMR
from paper_2508_05020_amd import workloads as W
from tests import _harness as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scale", [1.0, 2.0 ** 310, 2.0 ** -310])
@pytest.mark.parametrize("d,base,n", [(1, 8, 8), (1, 4096, 16), (2, 16, 16), (2, 512, 8), (3, 8, 8), (3, 12, 12), (3, 64, 4)])
def test_dt_is_exact(d, base, n, scale):
    import torch
    import paper_2508_05020_amd.amr as A
    cfg = W.AMRConfig(name="rate", dim=d, base_cells=base, patch_cells=[n], periodic=[True] * d,
                      max_patches=(base // n) ** d)
    h = A.Hierarchy(cfg)
    rng = np.random.default_rng(base + n)
    pids = [t["pid"] for t in h.patch_table()]
    dx = 1.0 / base
    worst = 0.0
    state = {}
    for pid in pids:
        box = (n + 8,) * d
        rho = rng.uniform(0.5, 2.0, box)
        m = [rho * rng.uniform(-1, 1, box) for _ in range(d)]
        if pid % 3 == 0:
            m[0] = np.zeros(box)
        p = rng.uniform(0.1, 1.0, box)
        ke = m[0] * (m[0] / rho)
        for j in range(1, d):
            ke = ke + m[j] * (m[j] / rho)
        u = np.stack([rho, *m, p / (cfg.gamma - 1.0) + 0.5 * ke]) * scale
        state[pid] = u
        u = H.interior(u, d)
        v = [u[1 + j] / u[0] for j in range(d)]
        ke = u[1] * v[0]
        for j in range(1, d):
            ke = ke + u[1 + j] * v[j]
        c = np.sqrt(cfg.gamma * ((cfg.gamma - 1.0) * (u[d + 1] - 0.5 * ke)) / u[0])
        s = np.abs(v[0]) + c
        for j in range(1, d):
            s = s + (np.abs(v[j]) + c)
        worst = max(worst, float(np.max(s / dx)))
    h.set_state(0, state)
    dt = h.compute_dt(0)
    assert float(dt.cpu()) == cfg.cfl / worst
    state[pids[-1]][(0,) + (4,) * d] = np.nan
    h.set_state(0, {pids[-1]: state[pids[-1]]})
    assert np.isnan(float(h.compute_dt(0).cpu()))
    h.close()
