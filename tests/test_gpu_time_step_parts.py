"""The CFL step where the ghost fill leaves more partial maxima of |U|^2 than have a place of their own in the
workspace: they then stand in a residual array until the step is formed."""
import numpy as np
import pytest
import torch

from gpu_util import print_case
from synth import make_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("grid", [(192, 96, 96), (40, 40, 700)])  # 2856 and 2824 of them, 2048 have a place
def test_cfl_step_of_many_partial_maxima(grid, precision):
    from paper_2603_11102_amd import GksSolver
    cfg = make_case("channel", grid=grid)
    q = cfg.q0.copy()
    q[3, -1, -1, -1] = 2.0  # the fastest cell is the last workgroup's
    cfg = cfg.with_(q0=q)
    print_case("many-maxima", grid=grid, precision=precision)
    s = GksSolver(cfg, precision=precision)
    h, c = min(cfg.dx, cfg.dy, cfg.dz), 1.0 / cfg.ma
    for _ in range(3):  # from the second step on the residual array holds the step before
        q = s.interior()
        u2 = float(((q[1:] ** 2).sum(0) / (cfg.rho_ref + q[0]) ** 2).max())
        s.step(1)
        # 1e-14: a few roundings of the sum, the quotient and the root
        assert abs(s.forces()["dt"] / (cfg.cfl * h / (np.sqrt(u2) + c)) - 1.0) < 1e-14
