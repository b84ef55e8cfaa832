"""Seams of the order-5 face passes where the library's own plan puts them (gks_face_plan): runs that go on from one tile
into the next and start their march anew there, in both launch schemes, both precisions and both FP64 tile heights,
whole fields against the oracle; and, at the sizes of the benchmark, sampled cells at the ends of marches and tiles.
Bars as in test_gpu_parity and test_gpu_fullsize."""
import ctypes as C

import numpy as np
import pytest
import torch

from gpu_util import oracle_dev, print_case, rel_errors, run_gpu, run_oracle
from sampling import box_ranges, box_reference, excluded, near_boundary, take_box
from synth import make_case

pytestmark = pytest.mark.gpu
AXES = ((0, 1, 2), (1, 0, 2), (2, 0, 1))  # (normal, t1, t2) of the x, y and z passes


def plan_of(s):
    out = (C.c_int * 11)()
    assert s.lib.gks_face_plan(s.ctx, None, None, out) == 0
    return {"side_by_side": out[0], "rows": out[1], "chunk": out[2::3], "seg_len": out[3::3], "n_wg": out[4::3]}


def marches(plan, d, n):
    """Marches (tile, first cell, end cell) of pass d on a grid n, workgroup by workgroup."""
    an, a1, a2 = AXES[d]
    tiles = -(-n[a1] // 16) * -(-n[a2] // plan["rows"])
    chunk, seg, n_wg = (plan[k][d] for k in ("chunk", "seg_len", "n_wg"))
    for w in range(n_wg):
        if seg == 0:
            c0 = w // tiles * chunk
            yield [(w % tiles, c0, min(c0 + chunk, n[an]))]
        else:
            lin, end, m = w * seg, min((w + 1) * seg, tiles * n[an]), []
            while lin < end:
                t, f0 = divmod(lin, n[an])
                f1 = min(n[an], f0 + end - lin)
                m.append((t, f0, f1))
                lin += f1 - f0
            yield m


@pytest.mark.parametrize("precision,grid,side_by_side,rows,axis", [
    ("fp32", (3, 161, 110), 0, 16, 0), ("fp32", (102, 3, 172), 0, 16, 1), ("fp32", (178, 169, 7), 0, 16, 2),
    ("fp32", (3, 101, 66), 1, 16, 0), ("fp32", (104, 3, 67), 1, 16, 1), ("fp32", (66, 105, 3), 1, 16, 2),
    ("fp64", (3, 151, 111), 0, 12, 0), ("fp64", (106, 5, 179), 0, 12, 1), ("fp64", (137, 170, 10), 0, 12, 2),
    ("fp64", (4, 55, 171), 0, 8, 0), ("fp64", (167, 3, 67), 0, 8, 1), ("fp64", (149, 117, 8), 0, 8, 2),
    ("fp64", (3, 116, 49), 1, 12, 0), ("fp64", (65, 4, 114), 1, 12, 1), ("fp64", (161, 38, 9), 1, 12, 2),
    ("fp32", (4, 3, 2100), 1, 16, 0), ("fp64", (4, 3, 2100), 1, 8, 1),
    ("fp64", (3, 25, 160), 1, 8, 0), ("fp64", (170, 3, 26), 1, 8, 1), ("fp64", (37, 166, 3), 1, 8, 2),
])
def test_runs_across_tiles_vs_oracle(precision, grid, side_by_side, rows, axis):
    cfg = make_case("channel", grid=grid)
    print_case("face-runs", precision=precision, grid=grid)
    s, _ = run_gpu(cfg, precision, 1)
    p = plan_of(s)
    assert (p["side_by_side"], p["rows"]) == (side_by_side, rows)
    assert any(len(m) > 1 for m in marches(p, axis, grid))  # some workgroup goes on into another tile
    o, _ = run_oracle(cfg, 1)
    err = rel_errors(s.interior(), oracle_dev(o.Q, cfg.rho_ref))
    assert max(err) < (1e-12 if precision == "fp64" else 1e-5), err


@pytest.mark.parametrize("case,precision,tol", [
    ("channel", "fp64", 1e-12),
    ("channel", "fp32", 2e-6),
    ("channel_tanh", "fp64", 1e-12),
    ("channel_tanh", "fp32", 2e-6),
    ("alm", "fp32", 2e-6),
])
def test_full_size_cells_at_the_plan_s_seams(case, precision, tol):
    from paper_2603_11102_amd import GksSolver
    cfg = make_case(case)
    rng = np.random.default_rng(12)
    q = cfg.q0.copy()
    q[1:] += 0.05 * rng.uniform(-1, 1, size=q[1:].shape)
    q[0] += 0.005 * rng.uniform(-1, 1, size=q[0].shape)
    cfg = cfg.with_(q0=q)
    n = (cfg.nx, cfg.ny, cfg.nz)
    print_case("full-size-seams", case=case, precision=precision, grid=n)
    s = GksSolver(cfg, precision=precision)
    p = plan_of(s)
    bad = excluded(cfg) | near_boundary(cfg)
    pick = []
    for d, (an, a1, a2) in enumerate(AXES):
        # first and last cells of marches, at the corners of their tile
        nt1, cells = -(-n[a1] // 16), set()
        crossing = [m for m in marches(p, d, n) if len(m) > 1] or list(marches(p, d, n))
        for m in crossing:
            for t, f0, f1 in m:
                for c in (f0, f1 - 1):
                    for e1 in (0, 15):
                        for e2 in (0, p["rows"] - 1):
                            x = [0, 0, 0]
                            x[an], x[a1], x[a2] = c, t % nt1 * 16 + e1, t // nt1 * p["rows"] + e2
                            if all(x[a] < n[a] for a in range(3)) and not bad[x[2], x[1], x[0]]:
                                cells.add((x[2], x[1], x[0]))
        cells = sorted(cells)
        assert cells, d
        pick += [np.array(cells[i]) for i in rng.choice(len(cells), size=min(5, len(cells)), replace=False)]
    boxes = []
    for cell in pick:
        rg = box_ranges(cfg, cell)
        boxes.append((rg, take_box(s.q, rg, pad=3)))
    s.step(1)
    dt = s.forces()["dt"]
    after = s.q[:, 3:-3, 3:-3, 3:-3]
    scale = torch.tensor([cfg.rho_ref, 1.0, 1.0, 1.0], dtype=torch.float64)
    for cell, (rg, b) in zip(pick, boxes):
        k, j, i = (int(c) for c in cell)
        err = ((after[:, k, j, i].to(torch.float64).cpu() - box_reference(cfg, b, rg, cell, dt)).abs() / scale).max()
        assert float(err) < tol, (cell, float(err))
