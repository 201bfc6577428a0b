"""Multi-step tiles (four steps per launch on small lattices): bit for bit the fused single steps,
for every geometry and equation of state, at sizes around the edges of each tile's range and with
every remainder of the step count; lattices narrower than the halo wrap several times. The fused
schedule itself is compared with the oracle elsewhere; equal bits need no tolerance."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

# 8x4 tiles up to 256 of them, 8x8 up to 256, 16x8 up to 512, then the two-step tiles
SIZES = [(5, 9), (128, 66), (129, 66), (128, 129), (129, 130), (257, 131), (300, 150), (512, 130),
         (513, 130)]


def _case(nx, ny, walls, eos):
    if eos == "piecewise":
        p = synth.paper_params(nx=nx, ny=ny, walls=walls, wall_force="modpsi")
        rl, rv, width = 500.0, 1.0, 4.0
    else:
        p = synth.base_params(nx=nx, ny=ny, walls=walls, wall_force="rho", tau_l=0.6, tau_v=1.0)
        rv, rl, width = 0.0008901265340675707, 0.445063267033785, 2.0
        p.update(rho_l=rl, rho_v=rv)
    r = 0.25 * min(nx, ny)
    centres = [(nx / 2.0, 0.5 if walls in (1, 2) else ny / 2.0)]
    rho = synth.droplet_rho(nx, ny, rl, rv, centres, [r], width=width, seed=nx + ny,
                            walls=walls in (1, 2))
    if walls == 3:
        solid = synth.pillar_mask(nx, ny, height=max(1, ny // 6))
        rho[solid != 0] = 0.0
        p.update(walls=3, ghost=0, solid=solid)
        return p, np.where(solid != 0, -1.0 if eos == "piecewise" else -0.05, 0.0), rho
    if walls == 0:
        return p, None, rho
    gw = synth.gw_smooth(nx, -0.05, 0.04, 3)
    gw[1] = gw[0][::-1]
    return p, gw, rho


@pytest.mark.parametrize("eos", ["cs", "piecewise"])
@pytest.mark.parametrize("walls", [0, 1, 2, 3])
def test_multi_step_bitwise_equals_single_steps(gpu, walls, eos):
    for nx, ny in SIZES:
        p, gw, rho = _case(nx, ny, walls, eos)
        one, many = gpu.Sim(p, gw, rho), gpu.Sim(p, gw, rho)
        one.set_schedule("fused")
        for n in (4, 5, 6, 11):
            one.step(n)
            many.step(n)
            a, b = one.f(), many.f()
            assert np.array_equal(a, b, equal_nan=True), (nx, ny, n, int((a != b).sum()))


def test_multi_step_recomputation_gives_the_same_gradient(gpu):
    """The segment states that the multi-step tiles recompute for the adjoint, against those of
    the two-step tiles (an output tile chosen by hand), for segments of every remainder."""
    p, gw, rho = _case(130, 70, 1, "cs")
    grads = []
    for schedule in (None, 39):
        sim = gpu.Sim(p, gw, rho)
        if schedule:
            sim.set_schedule(schedule)
        got = []
        for n, k in ((23, 9), (20, 6), (14, 7), (9, 8)):
            ws = sim.adjoint_workspace(n, k)
            sim.forward_ckpt(n, k, ws)
            sim.loss()
            got.append(sim.backward(n, k, ws).cpu().numpy())
        grads.append(got)
    for a, b in zip(*grads):
        assert np.isfinite(a).all() and np.abs(a).max() > 0 and np.array_equal(a, b)
