"""Two reverse steps per launch (small lattices, alone): gradients bit for bit those of the
ensemble's reverse sweep, which makes single ones, for lattices around the tile's edges and segments
of every remainder. The ensemble's gradients are compared with autograd and central differences
elsewhere; equal bits need no tolerance."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form,ratio", [("rho", 1.0), ("psi", 5.0), ("modpsi", 15.0)])
def test_two_reverse_steps_bitwise_equal_single_ones(gpu, form, ratio):
    cases = []
    for nx, ny in [(16, 10), (17, 27), (95, 42), (128, 66), (300, 150)]:
        p = synth.base_params(nx=nx, ny=ny, wall_force=form, rho_v=0.0008901265340675707,
                              rho_l=0.445063267033785)
        if ratio != 1.0:
            p.update(tau_l=0.6, tau_v=0.1 * ratio + 0.5)
        rho = synth.droplet_rho(nx, ny, p["rho_l"], p["rho_v"], [(nx / 2.0, 0.5)],
                                [0.3 * min(nx, ny)], seed=nx)
        gw = synth.gw_smooth(nx, -0.02, 0.02, 3)
        gw[1] = gw[0][::-1]
        cases.append((p, gw, rho))
    for n, k in ((13, 13), (16, 5), (7, 1), (12, 4)):
        b = gpu.Batch(*[list(c) for c in zip(*cases)])
        ws = b.adjoint_workspace(n, k)
        b.forward_ckpt(n, k, ws)
        b.loss()
        both = [g.cpu().numpy() for g in b.backward(n, k, ws)]
        for c, ref in zip(cases, both):
            s = gpu.Sim(*c)
            w = s.adjoint_workspace(n, k)
            s.forward_ckpt(n, k, w)
            s.loss()
            got = s.backward(n, k, w).cpu().numpy()
            assert np.isfinite(got).all() and np.abs(got).max() > 0
            assert np.array_equal(got, ref), (c[0]["nx"], n, k)


def test_checkpointed_forward_of_an_ensemble_can_be_captured(gpu):
    """A caller's graph capture of the checkpointed forward run (it has no host synchronisation):
    the replay leaves the state and the gradients of a run that was launched directly."""
    import torch

    p = synth.base_params(nx=96, ny=42, wall_force="modpsi", rho_v=0.0008901265340675707,
                          rho_l=0.445063267033785)
    rho = synth.droplet_rho(96, 42, p["rho_l"], p["rho_v"], [(48.0, 0.5)], [12.0], seed=3)
    gw = [synth.gw_smooth(96, -0.02, 0.02, k) for k in (3, 4)]
    ends = []
    for captured in (False, True):
        s = torch.cuda.Stream()
        b = gpu.Batch([p, p], gw, [rho, rho], tune={"tile": 1, "schedule": 2}, stream=s)
        ws = b.adjoint_workspace(11, 4)
        if captured:
            torch.cuda.synchronize()
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g, stream=s):
                b.forward_ckpt(11, 4, ws)
            with torch.cuda.stream(s):
                g.replay()
        else:
            b.forward_ckpt(11, 4, ws)
        b.loss()
        ends.append([b.f(0), b.f(1)] + [x.cpu().numpy() for x in b.backward(11, 4, ws)])
    for x, y in zip(*ends):
        assert np.isfinite(x).all() and np.array_equal(x, y)
