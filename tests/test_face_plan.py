"""The work split of the order-5 face launches, on the host: the split is the least one by its definition, and finding
it takes a small part of a context's initialisation."""
import ctypes as C
import random
import time

import pytest

from paper_2603_11102_amd import _lib as L
from test_workspace_sizes import config

SLOTS = (C.c_int * 2)(256, 256)


def plan(cfg, slots=SLOTS):
    out = (C.c_int * 11)()
    assert L.load().gks_face_plan(None, C.byref(cfg), slots, out) == L.GKS_OK
    return list(out)


def fewest(n, tiles, T, slots):
    """(workgroups, chunk, seg_len) of one direction whose marches take at most T face steps."""
    total, chunk = tiles * n, min(T - 2, n)
    best, seg = tiles * -(-n // chunk), 0
    for segs in range(1, (T - 2) // n + 3):
        ln = min(T - 2 * segs, total)
        if ln < 1:
            break
        wgs = -(-total // ln)
        if wgs >= best or wgs > slots:
            continue
        runs = [(w * ln, min(w * ln + ln, total)) for w in range(wgs)]
        if max(c1 - c0 + 2 * ((c1 - 1) // n - c0 // n + 1) for c0, c1 in runs) <= T:
            best, seg = wgs, ln
    return best, chunk, seg


def split(dirs, slots):
    T = 3  # the least T whose workgroups, padded to a multiple of 8 per direction, run at once
    def need(T):
        return sum((fewest(n, t, T, slots)[0] + 7) // 8 * 8 for n, t in dirs)
    hi = 3
    while need(hi) > slots:
        T, hi = hi + 1, 2 * hi
    while T < hi:
        mid = (T + hi) // 2
        if need(mid) <= slots:
            hi = mid
        else:
            T = mid + 1
    return hi, [fewest(n, t, hi, slots) for n, t in dirs]


def reference(grid, fp64, slots=256):
    best = None
    for rows, step in (((12, 6000.0), (8, 4600.0)) if fp64 else ((16, 4300.0),)):
        dirs = [(grid[a], -(-grid[b] // 16) * -(-grid[c] // rows)) for a, b, c in ((0, 1, 2), (1, 0, 2), (2, 0, 1))]
        txy, sxy = split(dirs[:2], slots)
        tz, sz = split(dirs[2:], slots)
        t3, s3 = split(dirs, slots - 8)
        cells = float(grid[0]) * grid[1] * grid[2]
        for scheme, t, s in ((0, step * (txy + tz) + 2000.0, sxy + sz),
                             (1, step * t3 + 4000.0 + (0.052 if fp64 else 0.039) * cells, s3)):
            if best is None or t < best[0]:
                best = (t, scheme, rows, s)
    return [best[1], best[2]] + [x for wgs, chunk, seg in best[3] for x in (chunk, seg, wgs)]


@pytest.mark.parametrize("precision", [L.GKS_FP32, L.GKS_FP64])
def test_split_is_the_least_by_definition(precision):
    rng = random.Random(11)
    grids = [(3, 3, 3), (16, 16, 12), (17, 33, 13), (192, 96, 96), (150, 77, 83), (4, 3, 2100), (128, 128, 128)]
    grids += [tuple(int(3 * 60.0 ** rng.random()) for _ in range(3)) for _ in range(60)]
    for g in grids:
        assert plan(config(g, precision)) == reference(g, precision == L.GKS_FP64), g


@pytest.mark.parametrize("grid,limit_us", [
    ((256, 256, 256), 60),      # gks_init itself takes about 150 us
    ((3, 512, 512), 60),
    ((2000, 2000, 3), 60),      # a march meets hundreds of tiles
])
def test_planning_time(grid, limit_us):
    cfg = config(grid, L.GKS_FP64)
    out = (C.c_int * 11)()
    f = L.load().gks_face_plan
    best = float("inf")
    for _ in range(200):
        t = time.perf_counter()
        f(None, C.byref(cfg), SLOTS, out)
        best = min(best, time.perf_counter() - t)
    assert best * 1e6 < limit_us
