"""Branches of the face kernels and their launch rules at the sizes and states where they can go wrong,
against the FP64 CPU oracle (bars as in test_gpu_parity: FP64 1e-12, FP32 1e-5, max norm per variable)."""
import pytest
import torch

from gpu_util import oracle_dev, print_case, rel_errors, run_gpu, run_oracle
from synth import make_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order", [5, 2])
@pytest.mark.parametrize("ma", [0.34, 0.6])
def test_kinetic_average_on_both_sides_of_its_series_range(ma, order):
    # |U| up to 1 and c = 1 / ma: sqrt(lambda) |U_n| reaches ma / sqrt(2) = 0.24, inside the series' range of
    # 1/4, and 0.42, where the field has Gauss points on both sides of it
    cfg = make_case("tgv", grid=(18, 14, 17)).with_(ma=ma, order=order)
    o, _ = run_oracle(cfg, 2)
    ref = oracle_dev(o.Q, cfg.rho_ref)
    for precision, bar in (("fp64", 1e-12), ("fp32", 1e-5)):
        print_case("kinetic", ma=ma, order=order, precision=precision)
        s, _ = run_gpu(cfg, precision, 2)
        err = rel_errors(s.interior(), ref)
        assert max(err) < bar, (precision, err)
        assert bool(torch.isfinite(s.interior()).all())


@pytest.mark.parametrize("case,grid", [
    ("tgv", (160, 78, 12)),      # x and y passes: the 12-row FP64 tile, z pass the 8-row one
    ("channel", (150, 70, 23)),  # z pass: the 12-row tile, t2 = 70 leaves ten rows of its last tile
])
def test_fp64_tile_heights_vs_oracle(case, grid):
    # the launch rule mixes the two FP64 tile heights over the directions at these sizes
    cfg = make_case(case, grid=grid)
    print_case("fp64-tiles", case=case, grid=grid)
    s, _ = run_gpu(cfg, "fp64", 1)
    o, _ = run_oracle(cfg, 1)
    err = rel_errors(s.interior(), oracle_dev(o.Q, cfg.rho_ref))
    assert max(err) < 1e-12, err


@pytest.mark.parametrize("precision,bar", [("fp64", 1e-12), ("fp32", 1e-5)])
@pytest.mark.parametrize("grid", [
    (3, 3, 3),      # one workgroup per direction, every cell within a stencil of two sides
    (24, 20, 18),   # the three directions in one launch
    (70, 66, 50),   # x and y passes in one launch, marches that cross tiles
])
def test_launch_schemes_vs_oracle(grid, precision, bar):
    cfg = make_case("channel", grid=grid)
    print_case("launch-scheme", grid=grid, precision=precision)
    s, _ = run_gpu(cfg, precision, 2)
    o, _ = run_oracle(cfg, 2)
    err = rel_errors(s.interior(), oracle_dev(o.Q, cfg.rho_ref))
    assert max(err) < bar, err


@pytest.mark.parametrize("precision,bar", [("fp64", 1e-12), ("fp32", 1e-5)])
@pytest.mark.parametrize("case,grid", [
    ("channel", (3, 3, 3)),       # fewer cells than the stencil reaches
    ("tgv", (33, 17, 9)),         # one cell past the 32 x 16 tile in x and y
    ("channel", (64, 32, 21)),    # whole tiles, walls at tile ends, several marches along z
    ("alm", (36, 18, 18)),        # inflow, outflow and slip ghost cells
])
def test_order2_stage_vs_oracle(case, grid, precision, bar):
    cfg = make_case(case, grid=grid).with_(order=2, rotor=None)
    print_case("order2-stage", case=case, grid=grid, precision=precision)
    s, _ = run_gpu(cfg, precision, 2)
    o, _ = run_oracle(cfg, 2)
    err = rel_errors(s.interior(), oracle_dev(o.Q, cfg.rho_ref))
    assert max(err) < bar, err


@pytest.mark.parametrize("grid", [
    (4, 3, 2100),   # more ghost-fill workgroups than a small workspace holds partial maxima: a pass of its own
    (40, 33, 30),   # partial maxima from the ghost fill, the step formed beside the face launch
    (70, 66, 50),   # the same with the step in a launch of its own
])
def test_time_step_and_bookkeeping_vs_oracle(grid):
    cfg = make_case("channel", grid=grid)
    print_case("time-step", grid=grid)
    s, outs = run_gpu(cfg, "fp64", 2)
    _, ref = run_oracle(cfg, 2)
    for n, (a, b) in enumerate(zip(outs, ref)):
        assert abs(a["dt"] - b["dt"]) < 1e-14 * b["dt"], (n, a["dt"], b["dt"])
        assert abs(a["t"] - b["t"]) < 1e-14 * b["t"]
        assert a["step"] == n + 1 and a["window_steps"] == n + 1
    s.step(3)
    assert s.forces()["step"] == 5


@pytest.mark.parametrize("precision,bar", [("fp64", 1e-12), ("fp32", 1e-5)])
@pytest.mark.parametrize("case,grid", [
    ("tgv", (26, 27, 4)),      # padded rows of one ghost-fill tile and of one tile and a cell; idle workgroups
    ("channel", (27, 26, 9)),  # the other way round
    ("alm", (54, 27, 27)),     # a row of one tile and a cell, every kind of open side
])
def test_ghost_fill_tiles_vs_oracle(case, grid, precision, bar):
    cfg = make_case(case, grid=grid).with_(rotor=None)
    print_case("ghost-tiles", case=case, grid=grid, precision=precision)
    s, _ = run_gpu(cfg, precision, 2)
    o, _ = run_oracle(cfg, 2)
    err = rel_errors(s.interior(), oracle_dev(o.Q, cfg.rho_ref))
    assert max(err) < bar, err
