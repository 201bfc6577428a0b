"""Marching strips (three steps per launch on lattices that fill the GPU): bit for bit the fused
single steps, for every geometry, equation of state and viscosity that takes them, at sizes with a
ragged last strip and segment, and for step counts with every remainder. The fused schedule itself
is compared with the oracle elsewhere; equal bits need no tolerance."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def _case(nx, ny, walls, eos, ratio, form):
    if eos == "piecewise":
        p = synth.paper_params(nx=nx, ny=ny, walls=walls, wall_force=form)
        rl, rv, width = 500.0, 1.0, 4.0
    else:
        p = synth.base_params(nx=nx, ny=ny, walls=walls, wall_force=form)
        rv, rl, width = 0.0008901265340675707, 0.445063267033785, 2.0
        p.update(rho_l=rl, rho_v=rv)
    if ratio != 1.0:
        p.update(tau_l=0.6, tau_v=0.1 * ratio + 0.5)
    r = 0.2 * min(nx, ny)
    # a droplet over the seam in x, and one on the bottom and top wall or over the seam in y
    # (its images on both sides, so that the field is continuous there)
    y0, y1 = (0.5, ny - 1.5) if walls else (0.0, float(ny))
    centres = [(nx / 2.0, y0), (nx / 2.0, y1), (0.0, ny / 2.0), (float(nx), ny / 2.0)]
    rho = synth.droplet_rho(nx, ny, rl, rv, centres, [r, r, r / 2, r / 2], width=width, seed=5,
                            walls=walls != 0)
    gw = synth.gw_smooth(nx, -0.05, 0.04, 3) if walls else None
    if gw is not None:
        gw[1] = gw[0][::-1]
    return p, gw, rho


SHAPES = [
    (1500, 1001, 0, "cs", 1.0, "psi"),          # periodic in y, 28 strips, the last 42 wide
    (1999, 777, 1, "cs", 5.0, "modpsi"),        # odd width: the last strip is one column
    (1345, 1201, 2, "piecewise", 1.0, "rho"),   # wet-node walls
    (1296, 1300, 1, "piecewise", 15.0, "psi"),  # whole strips only
    (160, 9000, 0, "cs", 1.0, "rho"),           # a tall lattice, three strips
]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: f"{s[0]}x{s[1]}-{s[2]}-{s[3]}-{s[4]:g}")
def test_marching_bitwise_equals_single_steps(gpu, shape):
    p, gw, rho = _case(*shape)
    one, many = gpu.Sim(p, gw, rho), gpu.Sim(p, gw, rho)
    one.set_schedule("fused")
    for n in (3, 4, 7, 8):
        one.step(n)
        many.step(n)
        assert one.current_step == many.current_step
        a, b = one.f(), many.f()
        assert np.isfinite(a).all()
        assert np.array_equal(a, b), (n, int((a != b).sum()))


def test_marching_ensemble_bitwise_equals_single_steps(gpu):
    """An ensemble of uneven lattices, both wall schemes, equations of state and viscosities in
    one work-list; 67 steps replay a captured graph and leave a remainder."""
    shapes = [(1024, 512, 1, "cs", 5.0, "modpsi"), (701, 903, 0, "cs", 1.0, "rho"),
              (640, 901, 2, "piecewise", 1.0, "psi"), (55, 40, 1, "cs", 1.0, "psi")]
    cases = [_case(*s) for s in shapes]
    b = gpu.Batch([c[0] for c in cases], [c[1] for c in cases], [c[2] for c in cases],
                  tune={"tile": 1, "schedule": 2})
    sims = [gpu.Sim(*c) for c in cases]
    for s in sims:
        s.set_schedule("fused")
    for n in (5, 67, 3):
        b.step(n)
        for i, s in enumerate(sims):
            s.step(n)
            assert np.array_equal(b.f(i), s.f()), (n, i)


def test_marching_state_round_trip(gpu):
    """The wall force of the wet-node scheme is part of the state that a marching launch leaves."""
    p, gw, rho = _case(1345, 1201, 2, "piecewise", 1.0, "modpsi")
    a = gpu.Sim(p, gw, rho)
    a.step(6)
    blob = a.save_state()
    b = gpu.Sim(p, gw, rho)
    b.load_state(blob)
    a.step(5)
    b.step(5)
    assert np.array_equal(a.f(), b.f())
