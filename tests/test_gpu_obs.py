"""Observables formed tile by tile (64 x 8 nodes and a ring in LDS): lattices around the edges of
those tiles, alone and as one ensemble, against the oracle and against each other.

Tolerances: extremes, velocities and mass are sums or extremes of FP64 values that agree with the
oracle's to 1e-12 of their size after a few steps (the step's own parity); the circle comes from
normal equations whose condition amplifies that by about the squared distance over the interface
width, 1e-8 at these sizes. A lattice alone and in an ensemble runs the same order of operations:
equal bits."""
import math

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu
KEYS = ("rho_min", "rho_max", "umax", "umax_liquid", "mass", "theta_deg", "xc", "yc", "r", "n_fit")
SIZES = [(63, 41), (64, 42), (65, 43), (128, 50), (129, 33), (40, 26)]


def _case(orc, nx, ny, walls):
    p = synth.base_params(nx=nx, ny=ny, walls=walls, wall_force="modpsi")
    q = orc.make_params(p)
    p = dict(p, rho_l=q.rho_l, rho_v=q.rho_v)
    y0 = ny / 2.0 if walls == 0 else 0.5
    rho = synth.droplet_rho(nx, ny, q.rho_l, q.rho_v, [(nx / 2.0, y0)], [0.3 * min(nx, ny)],
                            seed=nx, walls=walls != 0)
    gw = synth.gw_smooth(nx, 0.02, 0.02, seed=ny)
    return p, q, gw, rho


@pytest.mark.parametrize("walls", [0, 1, 2])
def test_observables_at_tile_edges(orc, gpu, walls):
    cases = [_case(orc, nx, ny, walls) for nx, ny in SIZES]
    b = gpu.Batch([c[0] for c in cases], [c[2] for c in cases], [c[3] for c in cases])
    b.step(6)
    planes = [2.0 + 0.25 * i for i in range(len(cases))]
    both, moved = b.observables(), b.observables(y_wall=planes)
    for i, (p, q, gw, rho) in enumerate(cases):
        s = gpu.Sim(p, gw, rho)
        s.step(6)
        alone, alone_moved = s.observables(), s.observables(y_wall=planes[i])
        for got, one in ((both[i], alone), (moved[i], alone_moved)):
            for k in KEYS:
                assert got[k] == one[k] or (math.isnan(got[k]) and math.isnan(one[k])), (i, k)
        o = orc.observables(q, gw if walls else None, s.f())
        for k in ("rho_min", "rho_max", "mass", "umax", "umax_liquid"):
            assert abs(alone[k] - o[k]) <= 1e-11 * max(abs(o[k]), 1e-3), (i, k, alone[k], o[k])
        assert alone["n_fit"] == o["n_fit"]
        for k in ("xc", "yc", "r"):
            assert abs(alone[k] - o[k]) <= 1e-7 * max(abs(o[k]), 1.0), (i, k, alone[k], o[k])


def test_nonfinite_nodes_are_counted(orc, gpu):
    """A state that leaves the EOS's domain: the count of nodes that are not finite equals the
    number of nodes whose velocity is not, alone and in an ensemble."""
    p, q, _, rho = _case(orc, 70, 37, 1)
    gw = synth.gw_uniform(70, -3.0)
    b = gpu.Batch([p, p], [gw, synth.gw_uniform(70, 0.05)], [rho, rho])
    s = gpu.Sim(p, gw, rho)
    for _ in range(60):
        b.step(1)
        s.step(1)
        o = s.observables(allow_nonfinite=True)
        if o["nonfinite"]:
            break
    both = b.observables(allow_nonfinite=True)
    assert o["nonfinite"] > 0 and both[0]["nonfinite"] == o["nonfinite"]
    assert both[1]["nonfinite"] == 0
    bad = ~np.isfinite(s.rho()[1:-1])
    assert o["nonfinite"] >= int(bad.sum())
