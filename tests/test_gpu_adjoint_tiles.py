"""The adjoint's tiles at sizes where their halos meet: one column or row past a tile, tiles with no whole
neighbour, marches of few faces. Held to the oracle's reverse mode (1e-10 in the scalings, 1e-9 in Q^0, as in
test_gpu_adjoint)."""
import numpy as np
import pytest
import torch

from gpu_util import print_case
from oracle import WenoControl, rotor_gradient, rotor_objective
from synth import make_case

pytestmark = pytest.mark.gpu
W = (1.0, 0.5)


@pytest.mark.parametrize("n", [18, 23, 33])  # 16 x 8 tiles: 16 + 2 and 2 x 8 + 2, 16 + 7 and 2 x 8 + 7, one past both
@pytest.mark.parametrize("exact", [False, True])
def test_adjoint_tiles_match_oracle_reference(n, exact):
    from paper_2603_11102_amd import GksSolver
    cfg = make_case("adjoint", grid=(n, n, n))
    scales = 1.0 + 0.1 * np.random.default_rng(3).standard_normal(cfg.rotor.n_act)
    print_case("adjoint-tiles", n=n, exact=exact)
    s = GksSolver(cfg, precision="fp64")
    sc = torch.as_tensor(scales, dtype=torch.float64, device="cuda").contiguous()
    s.set_rotor(cfg.rotor, scale=sc)
    s.set_checkpoints(1)
    s.step(1)
    g, gq = s.adjoint(1, W, want_field=True, exact=exact)
    _, go = rotor_gradient(cfg, scales, 1, W, frozen=not exact)
    assert float((g.cpu() - go).abs().max() / go.abs().max()) < 1e-10
    q0 = torch.tensor(cfg.q0).clone().requires_grad_(True)
    J, _ = rotor_objective(cfg, torch.tensor(scales), 1, W, None if exact else WenoControl("detach"), q0=q0)
    J.backward()
    for v in range(4):
        ref = q0.grad[v]
        assert float((gq[v].cpu() - ref).abs().max() / ref.abs().max()) < 1e-9, v


@pytest.mark.parametrize("bc", [
    ("outflow", "outflow", "noslip", "slip", "noslip", "noslip"),
    ("slip", "outflow", "periodic", "periodic", "outflow", "noslip"),
])
def test_adjoint_folds_every_side_kind(bc):
    # the transpose of the ghost fill with a different kind at either end of an axis, over two steps: the adjoint
    # fields change places between them, with ghost cells that have to stay zero
    from paper_2603_11102_amd import GksSolver
    n = 18
    cfg = make_case("adjoint", grid=(n, n, n)).with_(bc=bc)
    scales = 1.0 + 0.1 * np.random.default_rng(4).standard_normal(cfg.rotor.n_act)
    print_case("adjoint-folds", n=n, bc=bc)
    s = GksSolver(cfg, precision="fp64")
    sc = torch.as_tensor(scales, dtype=torch.float64, device="cuda").contiguous()
    s.set_rotor(cfg.rotor, scale=sc)
    s.set_checkpoints(2)
    s.step(2)
    g, gq = s.adjoint(2, W, want_field=True)
    _, go = rotor_gradient(cfg, scales, 2, W, frozen=True)
    assert float((g.cpu() - go).abs().max() / go.abs().max()) < 1e-10
    q0 = torch.tensor(cfg.q0).clone().requires_grad_(True)
    J, _ = rotor_objective(cfg, torch.tensor(scales), 2, W, WenoControl("detach"), q0=q0)
    J.backward()
    for v in range(4):
        ref = q0.grad[v]
        assert float((gq[v].cpu() - ref).abs().max() / ref.abs().max()) < 1e-9, v
