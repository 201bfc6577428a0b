"""Workspace sizes, without a GPU: what is reserved is what the kernels use."""
import ctypes as C

import pytest

import synth
import paper_1410_2569_amd as L

NX, NY = 1024, 512
PLANE = NX * NY * 8


@pytest.mark.parametrize("walls", [0, 1, 2, 3])
def test_an_ensemble_holds_populations_and_no_field(walls):
    """Ensembles form the pseudopotential tile by tile: per instance two buffers of nine planes (a
    mask adds G_w and the link words per node, 1.25 planes), and little beside them."""
    q = L.make_params(synth.base_params(nx=NX, ny=NY, walls=walls, ghost=int(walls != 3)))
    arr, n = (L.Params * 3)(q, q, q), C.c_size_t()
    assert L.lib().lbm_batch_workspace_size(arr, 3, None, C.byref(n)) == 0
    planes = n.value / (3 * PLANE) - (1.25 if walls == 3 else 0)
    assert 18 < planes < 18.2


@pytest.mark.parametrize("nsteps,K,states", [(1, 1, 1), (9, 1, 9), (9, 2, 5 + 2), (60, 8, 8 + 14),
                                             (7, 7, 1 + 12), (3, 7, 1 + 12)])
def test_a_segment_holds_its_states_without_the_checkpoint(nsteps, K, states):
    """One lattice: every checkpoint, two segments of K - 1 recomputed states (the first state of a
    segment is its checkpoint), and 26 planes of adjoint quantities."""
    q = L.make_params(synth.base_params(nx=NX, ny=NY))
    n = C.c_size_t()
    assert L.lib().lbm_adjoint_workspace_size(C.byref(q), nsteps, K, C.byref(n)) == 0
    planes = n.value / PLANE
    assert 9 * states + 26 < planes < 9 * states + 26.2
