"""The adjoint workspace is as large as its size query says and no larger part of it is written: the
bytes behind it stay as they were, and the gradients do not depend on what it held before. One
lattice and an ensemble, segments of every remainder, on a lattice of the multi-step tiles and on
one of the two-step tiles."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu
TAIL = 1 << 20


def _guarded(ws, byte):
    import torch

    buf = torch.full((ws.numel() + TAIL,), byte, dtype=torch.uint8, device="cuda")
    return buf, buf[:ws.numel()]


@pytest.mark.parametrize("nx,ny", [(95, 42), (700, 390)])
@pytest.mark.parametrize("n,k", [(5, 1), (7, 2), (11, 4), (13, 6), (6, 9)])
def test_nothing_behind_the_workspace_is_written(gpu, nx, ny, n, k):
    import torch

    p = synth.base_params(nx=nx, ny=ny, wall_force="modpsi", rho_v=0.0008901265340675707,
                          rho_l=0.445063267033785)
    rho = synth.droplet_rho(nx, ny, p["rho_l"], p["rho_v"], [(nx / 2.0, 0.5)], [0.3 * ny], seed=3)
    gw = [synth.gw_smooth(nx, -0.02, 0.02, s) for s in (3, 4)]
    grads = []
    for byte in (0, 255):  # zeros, NaN
        for make in (lambda: gpu.Sim(p, gw[0], rho), lambda: gpu.Batch([p, p], gw, [rho, rho])):
            s = make()
            buf, ws = _guarded(s.adjoint_workspace(n, k), byte)
            torch.cuda.synchronize()
            s.forward_ckpt(n, k, ws)
            s.loss()
            g = s.backward(n, k, ws)
            torch.cuda.synchronize()
            assert bool((buf[ws.numel():] == byte).all())
            grads.append((g[0] if isinstance(g, list) else g).cpu().numpy())
    assert np.isfinite(grads[0]).all() and np.abs(grads[0]).max() > 0
    for g in grads[1:]:
        assert np.array_equal(g, grads[0])
