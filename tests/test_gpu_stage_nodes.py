"""The node/edge phases of the stage kernel at the edges of every tile (GPU):
L(U) of rough random states, whose interpolated pressure is not positive at
many edges (the two-node fallback), against the oracle for every admissible
tile variant and both primitive schemes.

Tolerance: an edge value is about 60 operations on values whose differences
are of the values' own size (random states: no cancellation beyond a factor of
about ten), L(U) a sum of 4 d edge fluxes; 100 operations times 2^-53 times a
factor of ten is 1e-13, and the bound is the parity bar 1e-12.
"""
import numpy as np
import pytest

from oracle import euler
from oracle.solver import OracleAMR
from paper_2508_05020_amd import workloads as W
from tests import _harness as H


def _rough(o, seed):
    """rho and p log-uniform over [1e-3, 1], |u| <= 0.1, one level, periodic."""
    rng = np.random.default_rng(seed)

    def gen(pts):
        shape = pts[0].shape
        return (10.0 ** rng.uniform(-3, 0, shape), [rng.uniform(-0.1, 0.1, shape) for _ in pts],
                10.0 ** rng.uniform(-3, 0, shape))
    for k in o.forest.keys():
        o.set_initial(k, gen)


def _config(d, n):
    return W.AMRConfig(name=f"rough{d}", dim=d, base_cells=2 * n, patch_cells=[n],
                       periodic=[True] * d, max_patches=64)


SIZES = [(1, 8), (1, 16), (2, 8), (2, 16), (2, 24), (3, 4), (3, 8), (3, 12)]


@pytest.mark.parametrize("d,n", SIZES)
def test_rough_states_reach_the_fallback(d, n):
    """The states of the next test have edges whose interpolated p is not positive."""
    cfg = _config(d, n)
    o = OracleAMR(cfg)
    _rough(o, 77)
    p = euler.primitives(o.canvas(0, 0)[0], d, cfg.gamma)[2]
    v = [np.roll(p, 2 - k, axis=-1) for k in range(5)]
    left = euler.weno5js(*v, cfg.weno_eps)
    share = float(np.mean(left <= 0.0))
    assert 0.0 < share < 0.5, share


@pytest.mark.gpu
@pytest.mark.parametrize("scheme", ["weno", "central"])
@pytest.mark.parametrize("d,n", SIZES)
def test_rhs_of_rough_states_every_tile(d, n, scheme):
    import paper_2508_05020_amd.amr as A
    cfg = _config(d, n)
    o = OracleAMR(cfg, scheme=scheme)
    _rough(o, 77)
    o.fill_ghosts(0)
    ref = o.rhs(0)
    dt = o.compute_dt(0)
    done = 0
    for v in range(11):
        h = A.Hierarchy(cfg, scheme=H.SCHEMES[scheme])
        pid_of, _ = H.mirror(o, h, bufs=(0,))
        try:
            h.set_tile_variant(v)
        except A.AMRError:
            h.close()
            continue
        got = H.tensor_patches(h, h.rhs(0), pid_of)
        err = H.rhs_error({k: H.interior(got[k], d) for k in ref}, ref, o.U[0], list(ref), d, dt)
        assert err <= H.TOL, (v, err)
        done += 1
        h.close()
    assert done >= 1
