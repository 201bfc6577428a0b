"""A caller's graph capture of an ensemble's steps, whatever the ensemble ran before and however many
steps: the capture itself runs nothing (a graph of the ensemble's own launched into it would run at
once and be missing from the replays), and each replay does the steps, to the bits of a run that was
launched directly."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


CASES = [  # lattices, steps (replayed from the ensemble's own graphs, or fewer), schedule
    (1024, 512, 3, 60, 2), (1024, 512, 3, 63, 2), (1024, 512, 3, 32, 2), (96, 48, 2, 64, 2),
    (96, 48, 2, 130, 2), (96, 48, 2, 64, 0), (96, 48, 2, 10, 1), (96, 48, 2, 11, 1)]


@pytest.mark.parametrize("nx,ny,count,n,schedule", CASES)
def test_steps_of_an_ensemble_can_be_captured(gpu, nx, ny, count, n, schedule):
    import torch

    p = synth.base_params(nx=nx, ny=ny, wall_force="modpsi", rho_v=0.0008901265340675707,
                          rho_l=0.445063267033785)
    rho = synth.droplet_rho(nx, ny, p["rho_l"], p["rho_v"], [(nx / 2.0, 0.5)], [0.3 * ny], seed=3)
    gw = [synth.gw_smooth(nx, -0.02, 0.02, k) for k in range(count)]

    def ensemble():
        s = torch.cuda.Stream()
        b = gpu.Batch([p] * count, gw, [rho] * count, tune={"tile": 1, "schedule": schedule},
                      stream=s)
        b.step(n)
        b.step(n)  # both parities of the buffers have run
        return b, s

    b, s = ensemble()
    torch.cuda.synchronize()
    before = b.ws.clone()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        b.step(n)
    torch.cuda.synchronize()
    assert torch.equal(b.ws, before)
    ref, _ = ensemble()
    for _ in range(3):  # from the same state, with work of its own between the replays
        b.ws.copy_(before)
        torch.cuda.synchronize()
        with torch.cuda.stream(s):
            g.replay()
        torch.cuda.synchronize()
    ref.step(n)
    assert b.current_step == ref.current_step == 3 * n
    for i in range(count):
        f = ref.f(i)
        assert np.isfinite(f).all() and np.array_equal(b.f(i), f)
