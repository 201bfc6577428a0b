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
