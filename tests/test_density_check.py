"""The check of the initial densities, without a GPU: every fluid node is looked at and no solid
node. (The size of the workspace is checked after them, before any HIP call: with one byte too few,
accepted densities give LBM_E_SIZE and refused ones LBM_E_INVAL.)"""
import ctypes as C
import math

import numpy as np
import pytest

import synth
import paper_1410_2569_amd as L

NX, NY = 37, 11
EINVAL, ESIZE = -1, -2


def _create(walls, rho, solid=None):
    q = L.make_params(synth.base_params(nx=NX, ny=NY, walls=walls, ghost=int(walls != 3)))
    dp = C.POINTER(C.c_double)
    h, ws, size = C.c_void_p(), C.c_void_p(256), L.workspace_size(q) - 1
    gw = np.zeros((NY if walls == 3 else 2, NX))
    g, r = gw.ctypes.data_as(dp), rho.ctypes.data_as(dp)
    if walls == 3:
        return L.lib().lbm_create_masked(C.byref(q), solid.ctypes.data_as(C.c_void_p), g, r, ws,
                                         size, None, C.byref(h))
    return L.lib().lbm_create(C.byref(q), g, r, ws, size, None, C.byref(h))


@pytest.mark.parametrize("walls", [0, 1, 2, 3])
@pytest.mark.parametrize("value", [0.0, -0.1, math.nan, math.inf, 0.7])
def test_every_fluid_density_and_no_solid_one(walls, value):
    solid = np.zeros((NY, NX), np.uint8)
    if walls == 3:
        solid[2:5, 7:30:3] = 1
        solid[:, 0] = 1
    elif walls:
        solid[0] = solid[-1] = 1
    good = np.where(solid != 0, value, 0.3)
    assert _create(walls, good, solid) == ESIZE
    fluid = np.argwhere(solid == 0)
    for y, x in [fluid[0], fluid[-1], fluid[len(fluid) // 2], fluid[NX - 1], fluid[-NX]]:
        bad = good.copy()
        bad[y, x] = value
        assert _create(walls, bad, solid) == EINVAL, (y, x)


def test_a_lattice_of_solid_nodes_alone_is_refused():
    assert _create(3, np.full((NY, NX), 0.3), np.ones((NY, NX), np.uint8)) == EINVAL
