"""FP32 second-order variant: what is small beside a workgroup's momenta keeps its own digits.

A momentum that doubles from cell to cell away from two no-slip walls, 2^-15 at the walls and 1 in the core, at
uniform density: the exact scheme reduces to the diffusion of that momentum, every other term cancels bit for bit
between the faces of a cell. FP32 is held against FP64 from the same field, cell by cell relative to the cell's own
value. With nu = mu dt / (rho h^2) = 0.1 and neighbours of 2 m and m / 2 a step's increment is at most 0.15 m; each
flux (difference, spacing, viscosity, reciprocal, product) carries 8 roundings u = 2^-24 and the divergence 5 more, so a
step adds at most 2 u m, and errors handed on by the neighbours grow by 1 + 3 nu a step: 16 u after four steps, one more
for the stored value. The bar is 24 u. A momentum held as its deviation from a value of the core would be
off by 2^-25 absolutely, 2^-10 of the wall cell's momentum."""
import numpy as np
import pytest
import torch

from gpu_util import print_case
from synth import make_case
from synth.cases import tanh_faces

pytestmark = pytest.mark.gpu
U = 2.0 ** -24


@pytest.mark.parametrize("stretched", [False, True])
@pytest.mark.parametrize("axis", [0, 1, 2])
def test_wall_momentum_keeps_its_own_digits(axis, stretched):
    from paper_2603_11102_amd import GksSolver
    n = [10, 18, 6]
    n[axis] = 32
    k = np.arange(32)
    prof = 2.0 ** (np.minimum(k, 31 - k) - 15.0)
    along = (axis + 1) % 3  # the tangential momentum that carries the shear
    q = np.zeros((4, n[2], n[1], n[0]))
    q[0] = 1.0
    shape = [1, 1, 1]
    shape[2 - axis] = 32
    q[1 + along] = prof.reshape(shape)
    faces = [None, None, None]
    if stretched:
        faces[axis] = tanh_faces(32) + 1.0
        hmin = float(np.diff(faces[axis]).min())
    else:
        hmin = 2.0 / 32
    lens = [0.1 * a for a in n]
    lens[axis] = 2.0
    bc = ["periodic"] * 6
    bc[2 * axis] = bc[2 * axis + 1] = "noslip"
    dt = 0.3 * hmin / 11.0  # |U| <= 1, c = 1 / ma = 10
    cfg = make_case("channel", grid=(8, 8, 8)).with_(
        nx=n[0], ny=n[1], nz=n[2], x0=0.0, y0=0.0, z0=0.0, lx=lens[0], ly=lens[1], lz=lens[2], bc=tuple(bc), order=2,
        ma=0.1, mu=0.1 * hmin * hmin / dt, cfl=0.0, dt_fixed=dt, body_force=(0.0, 0.0, 0.0), q0=q,
        faces=tuple(faces) if stretched else None)
    print_case("order2-shear", axis=axis, stretched=stretched)
    f = {}
    for p in ("fp32", "fp64"):
        s = GksSolver(cfg, precision=p)
        s.step(4)
        f[p] = s.interior()
        s.close()
    ref = f["fp64"][1 + along]
    assert float((ref - torch.tensor(q[1 + along])).abs().max()) > 1e-3  # the layer has diffused
    err = ((f["fp32"][1 + along] - ref) / ref).abs().max()
    print(f"[order2-shear] axis {axis} stretched {stretched}: worst relative error {float(err) / U:.1f} u")
    assert float(err) < 24 * U


@pytest.mark.parametrize("axis", [0, 1, 2])
def test_density_of_a_stream_between_walls_keeps_its_own_digits(axis):
    # A stream of 0.27 with disturbances of 1e-3 towards slip walls, whose ghost cells mirror it to -0.27: away from
    # the walls the density changes by the disturbances' divergence only, and FP32 must round at their size, not at the
    # stream's. A mass flux taken as its deviation from a constant near 0.27 carries 4 roundings of 1e-3 in its products
    # and, with a = sqrt(lambda) U = 0.019, u a on the difference of aL and aR: (0.27 * 0.56 a + 2 a^2 / (2 sqrt(pi
    # lambda))) u = 0.006 u; a step's density takes two faces times dt / h = 0.03: 6e-4 u. The bar is four times that;
    # whole mass fluxes round at 0.27 / 4 and more, 1e-2 u here.
    from paper_2603_11102_amd import GksSolver
    n, h = [20, 18, 6], 0.1
    n[axis] = 24
    q = np.zeros((4, n[2], n[1], n[0]))
    q[0] = 1.0
    # both precisions start from the same field
    q[1 + axis] = (0.27 + 1e-3 * np.random.default_rng(6).uniform(-1, 1, size=q[1].shape)).astype(np.float32)
    cfg = make_case("channel", grid=(8, 8, 8)).with_(
        nx=n[0], ny=n[1], nz=n[2], x0=0.0, y0=0.0, z0=0.0, lx=h * n[0], ly=h * n[1], lz=h * n[2], order=2, ma=0.1, mu=1e-3,
        bc=tuple("slip" if a // 2 == axis else "periodic" for a in range(6)), cfl=0.0, dt_fixed=0.03 * h,
        body_force=(0.0, 0.0, 0.0), q0=q)
    print_case("order2-stream", axis=axis)
    f = {}
    for p in ("fp32", "fp64"):
        s = GksSolver(cfg, precision=p)
        s.step(1)
        f[p] = s.interior()[0].narrow(2 - axis, 6, 12)  # a step reaches four cells
        s.close()
    err = float((f["fp32"] - f["fp64"]).abs().max())
    print(f"[order2-stream] worst density error {err / U:.2e} u, density deviation up to {float(f['fp64'].abs().max()):.1e}")
    assert err < 2.5e-3 * U
