"""Workspace sizes that programs may have stored: a caller's buffer of such a size stays large enough."""
import ctypes as C

import pytest

from paper_2603_11102_amd import _lib as L


def config(grid, precision, order=5, max_act=0, max_ibm=0):
    c = L.gks_config()
    c.nx, c.ny, c.nz = grid
    c.precision = precision
    c.lx = c.ly = c.lz = 1.0
    c.ma, c.u_ref, c.rho_ref, c.mu, c.cfl = 0.1, 1.0, 1.0, 1e-3, 0.5
    c.ibm_iters, c.order, c.max_act, c.max_ibm = 3, order, max_act, max_ibm
    return c


@pytest.mark.parametrize("grid,precision,order,max_act,max_ibm,stored", [
    ((16, 16, 16), L.GKS_FP32, 5, 0, 0, 681472),
    ((24, 20, 18), L.GKS_FP64, 5, 96, 0, 2102272),
    ((192, 96, 96), L.GKS_FP32, 5, 0, 0, 231197696),    # more partial maxima of |U| than the room of their own
    ((192, 96, 96), L.GKS_FP64, 5, 0, 0, 292471808),
    ((192, 96, 96), L.GKS_FP32, 2, 0, 0, 231197696),
    ((150, 77, 83), L.GKS_FP32, 5, 0, 0, 127058432),
    ((384, 192, 192), L.GKS_FP32, 5, 192, 0, 1830170624),
    ((512, 256, 256), L.GKS_FP32, 5, 192, 26000, 4443650816),
    ((4, 3, 2100), L.GKS_FP64, 5, 0, 0, 16382208),
    ((40, 40, 700), L.GKS_FP64, 5, 0, 0, 205570816),
    ((128, 128, 128), L.GKS_FP64, 5, 96, 0, 345504256),
])
def test_context_workspace_fits_a_stored_size(grid, precision, order, max_act, max_ibm, stored):
    need = L.load().gks_workspace_bytes(C.byref(config(grid, precision, order, max_act, max_ibm)))
    assert 0 < need <= stored


@pytest.mark.parametrize("grid,n_act,stored", [
    ((128, 128, 128), 96, 2587484672),
    ((48, 48, 48), 48, 146426368),
    ((20, 120, 20), 96, 70588416),
    ((17, 9, 9), 6, 2835200),       # one cell past a tile, nine of two tiles' sixteen rows
    ((16, 8, 9), 6, 2465024),
    ((3, 24, 3), 0, 948224),        # narrower than a tile
    ((9, 3, 3), 6, 420352),
    ((3, 3, 187), 3, 6529024),
])
def test_adjoint_workspace_fits_a_stored_size(grid, n_act, stored):
    need = L.load().gks_adjoint_workspace_bytes(C.byref(config(grid, L.GKS_FP64, 5, 96)), n_act)
    assert 0 < need <= stored
