"""Which launches a schedule makes, counted as the nodes of a captured graph: the default takes four
steps per launch on small lattices and three on large ones; an output tile (32 + t) takes two; going
back to schedule 2 (the default) takes as many as a new context."""
import ctypes as C

import pytest

import synth

pytestmark = pytest.mark.gpu


def _launches(gpu, sim, stream, steps):
    import torch

    g = torch.cuda.CUDAGraph(keep_graph=True)
    torch.cuda.synchronize()
    with torch.cuda.graph(g, stream=stream):
        sim.step(steps)
    n = C.c_size_t()
    count = gpu.lib().hipGraphGetNodes  # of the runtime that the library is linked with
    count.argtypes, count.restype = [C.c_void_p, C.c_void_p, C.c_void_p], C.c_int
    assert count(g.raw_cuda_graph(), None, C.byref(n)) == 0
    return n.value


@pytest.mark.parametrize("nx,ny,default", [(120, 60, 3), (1500, 900, 4), (700, 400, 6)])
def test_schedule_2_is_the_default_again(gpu, nx, ny, default):
    import torch

    p = synth.base_params(nx=nx, ny=ny, rho_v=0.0008901265340675707, rho_l=0.445063267033785)
    rho = synth.droplet_rho(nx, ny, p["rho_l"], p["rho_v"], [(nx / 2.0, 0.5)], [0.2 * ny], seed=1)
    s = torch.cuda.Stream()
    sim = gpu.Sim(p, synth.gw_uniform(nx, 0.05), rho, stream=s)
    assert _launches(gpu, sim, s, 12) == default
    for tile in (0, 7):
        sim.set_schedule(32 + tile)
        assert _launches(gpu, sim, s, 12) == 6
        sim.set_schedule("fused")
        assert _launches(gpu, sim, s, 12) == 12
        sim.set_schedule("two_step")
        assert _launches(gpu, sim, s, 12) == default
