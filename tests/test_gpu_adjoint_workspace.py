"""The adjoint on grids narrower than a tile of its kernel, whose slab keeps only the columns that cells of the domain
reach: the gradient against the oracle's reverse mode (bars as in test_gpu_adjoint) and the bytes past the
workspace untouched."""
import ctypes as C
import dataclasses

import numpy as np
import pytest
import torch

from gpu_util import print_case
from oracle import WenoControl, rotor_gradient, rotor_objective
from synth import make_case

pytestmark = pytest.mark.gpu
W = (1.0, 0.5)
GUARD = 1 << 16


@pytest.mark.parametrize("exact", [False, True])
@pytest.mark.parametrize("grid", [
    (9, 9, 9),      # one tile of nine columns, two of eight and one row
    (17, 10, 12),   # one column past a tile
    (12, 16, 9),    # a whole tile in one direction, part of one in the others
])
def test_adjoint_of_narrow_grids(grid, exact):
    from paper_2603_11102_amd import GksSolver
    base = make_case("adjoint", grid=(18, 18, 18))
    h = base.lx / 18
    lens = [h * a for a in grid]
    # the points within 1.1 cells of the hub, their spheres of 3 eps within 3.6: inside nine cells
    r = np.array([0.5, 1.1]) * h
    rotor = dataclasses.replace(base.rotor, n_per_blade=2, hub=tuple(0.5 * a for a in lens), radius=1.3 * h, r=r,
                                chord=np.full(2, 0.1 * h), twist=np.array([0.2, 0.1]), width=np.full(2, 0.6 * h),
                                eps=0.8 * h, omega=0.7 / h)
    rng = np.random.default_rng(8)
    q = np.zeros((4, grid[2], grid[1], grid[0]))
    q[0], q[1] = 1.0, 1.0
    q[1:] += 0.05 * rng.uniform(-1, 1, size=q[1:].shape)
    cfg = base.with_(nx=grid[0], ny=grid[1], nz=grid[2], lx=lens[0], ly=lens[1], lz=lens[2], rotor=rotor, q0=q)
    scales = 1.0 + 0.1 * rng.standard_normal(rotor.n_act)
    print_case("adjoint-narrow", grid=grid, exact=exact)
    s = GksSolver(cfg, precision="fp64")
    s.set_rotor(rotor, scale=torch.as_tensor(scales, dtype=torch.float64, device="cuda").contiguous())
    s.set_checkpoints(2)
    s.step(2)
    need = s.lib.gks_adjoint_workspace_bytes(C.byref(s.c_cfg), s.n_act)
    s._adj_ws = torch.full((need + 256 + GUARD,), 0xA5, dtype=torch.uint8, device="cuda")
    g, gq = s.adjoint(2, W, want_field=True, exact=exact)
    end = -s._adj_ws.data_ptr() % 256 + need
    assert bool((s._adj_ws[end:] == 0xA5).all())
    _, go = rotor_gradient(cfg, scales, 2, W, frozen=not exact)
    assert float((g.cpu() - go).abs().max() / go.abs().max()) < 1e-10
    q0 = torch.tensor(cfg.q0).clone().requires_grad_(True)
    J, _ = rotor_objective(cfg, torch.tensor(scales), 2, W, None if exact else WenoControl("detach"), q0=q0)
    J.backward()
    for v in range(4):
        ref = q0.grad[v]
        assert float((gq[v].cpu() - ref).abs().max() / ref.abs().max()) < 1e-9, v
