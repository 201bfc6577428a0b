"""Large results on their way to the host: sizes around the limit from which they go through pinned
buffers and around the buffers' own, several readers at once, and a reader beside another stream's
work. Reference: torch's copy of the same device memory (the library forms a result densely in the
idle population buffer of the workspace before it copies it); equal bytes."""
import threading

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def _sim(gpu, nx, ny, seed=1, stream=None):
    p = synth.base_params(nx=nx, ny=ny, rho_v=0.0008901265340675707, rho_l=0.445063267033785)
    rho = synth.droplet_rho(nx, ny, p["rho_l"], p["rho_v"], [(nx / 2.0, 0.5)],
                            [0.2 * min(nx, ny)], seed=seed)
    return gpu.Sim(p, synth.gw_uniform(nx, 0.05), rho, stream=stream)


def _on_device(sim, buffer, n):
    """n doubles of population buffer 0 or 1 of the workspace, by torch."""
    plane = sim.ny * ((sim.nx + 31) // 32 * 32)
    o = buffer * ((9 * plane * 8 + 255) // 256 * 256)
    return sim.ws[o:o + 8 * n].cpu().numpy().view(np.float64)


# one row short of 8 MiB, 8 MiB (two buffers), one row and some columns more, three buffers less and
# more one row, and a size that nothing divides
@pytest.mark.parametrize("nx,ny", [(1024, 1023), (1024, 1024), (1024, 1025), (1027, 1024),
                                   (1024, 1535), (1024, 1537), (1283, 1021)])
def test_densities_around_the_buffers_sizes(gpu, nx, ny):
    sim = _sim(gpu, nx, ny)
    rho = sim.rho()
    assert rho[ny // 4, nx // 2] > 0
    assert np.array_equal(rho.ravel(), _on_device(sim, 1, nx * ny))


def test_populations_and_saved_state(gpu):
    sim = _sim(gpu, 1024, 300)
    f = sim.f()
    assert np.array_equal(f.ravel(), _on_device(sim, 1, f.size))
    blob = np.frombuffer(sim.save_state(), dtype=np.float64, offset=32)  # not page-aligned
    assert np.array_equal(blob, _on_device(sim, 0, f.size))


def test_more_readers_than_buffers(gpu):
    """Seven threads, each with a lattice of its own: more than the buffers that are kept."""
    import torch

    sims = [_sim(gpu, 640, 251, seed=k, stream=torch.cuda.Stream()) for k in range(7)]
    want = [s.f() for s in sims]
    bad = []

    def read(k):
        for _ in range(4):
            if not np.array_equal(sims[k].f(), want[k]):
                bad.append(k)

    th = [threading.Thread(target=read, args=(k,)) for k in range(len(sims))]
    for t in th:
        t.start()
    for t in th:
        t.join()
    assert not bad
    for k in (0, 6):
        assert np.array_equal(want[k].ravel(), _on_device(sims[k], 1, want[k].size))


def test_a_read_waits_for_its_own_stream_only(gpu):
    """While another stream still has some 150 ms of queued steps, a read-out of 83 MB (8 ms)
    returns: with pinned buffers yet to be made, and with those that are kept."""
    import torch

    mine, other = torch.cuda.Stream(), torch.cuda.Stream()
    a, b = _sim(gpu, 1200, 960, stream=mine), _sim(gpu, 2048, 1024, stream=other)
    want = a.f()
    for k in range(4):
        if k % 2 == 0:
            gpu.release_host_buffers()
        b.step(30)
        torch.cuda.synchronize()
        done = torch.cuda.Event()
        b.step(5100)
        done.record(other)
        got = a.f()
        assert not done.query()
        assert np.array_equal(got, want)
        torch.cuda.synchronize()
