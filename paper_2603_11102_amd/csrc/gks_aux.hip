// gks_aux.hip -- ghost cells, CFL time step, step bookkeeping and FP64 diagnostics.
//
// Boundary ghost cells (three layers) follow the boundary conditions named in Section 4:
// periodic; no-slip isothermal wall (mirror, rho even, all momenta odd); slip / symmetry wall
// (mirror, normal momentum odd); inflow with prescribed velocity and the density from the outgoing
// isothermal Riemann invariant U -+ C ln rho; zero-gradient outflow. Axes are filled x, then y, then z
// over the full padded extent of the other axes, so edges and corners are consistent.
// Time step: dt = CFL min(dx, dy, dz) / (|U|_max + C), C = sqrt(1/(2 lambda)) (Section 2).
#include <algorithm>

#include "gks.h"
#include "gks_internal.h"

namespace gks {

struct GhostArgs {
    int axis, n, np1, np2;
    long long st_a, st_1, st_2;
    int bc_lo, bc_hi;
    double u_in[3];
    double c, rho_ref;
};

template <typename real>
__global__ void ghost_kernel(Field4<real> f, GhostArgs g) {
    const long long per_side = 3LL * g.np1 * g.np2;
    const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= 2 * per_side) return;
    const int side = (int)(t / per_side);
    long long r = t % per_side;
    const int layer = (int)(r / ((long long)g.np1 * g.np2));
    r %= (long long)g.np1 * g.np2;
    const int p1 = (int)(r % g.np1), p2 = (int)(r / g.np1);
    const long long base = (long long)p1 * g.st_1 + (long long)p2 * g.st_2;
    // padded index along the axis: interior cell i sits at i + 3
    const int gi = side == 0 ? (2 - layer) : (g.n + 3 + layer);
    const int kind = side == 0 ? g.bc_lo : g.bc_hi;
    const long long dst = base + (long long)gi * g.st_a;
    int src_i;
    if (kind == 0) src_i = side == 0 ? (g.n - 1 - layer) : layer;                      // periodic
    else if (kind == 1 || kind == 2) src_i = side == 0 ? layer : (g.n - 1 - layer);    // mirror
    else src_i = side == 0 ? 0 : g.n - 1;                                              // adjacent cell
    const long long src = base + (long long)(src_i + 3) * g.st_a;
    if (kind == 0 || kind == 4) {
#pragma unroll
        for (int v = 0; v < 4; ++v) f.v[v][dst] = f.v[v][src];
    } else if (kind == 1) {
        f.v[0][dst] = f.v[0][src];
#pragma unroll
        for (int v = 1; v < 4; ++v) f.v[v][dst] = -f.v[v][src];
    } else if (kind == 2) {
#pragma unroll
        for (int v = 0; v < 4; ++v) f.v[v][dst] = (v == 1 + g.axis) ? -f.v[v][src] : f.v[v][src];
    } else {  // inflow
        const double rp = (double)f.v[0][src];
        const double rho_i = g.rho_ref + rp;
        const double un = (double)f.v[1 + g.axis][src] / rho_i;
        const double x = side == 0 ? (g.u_in[g.axis] - un) / g.c : (un - g.u_in[g.axis]) / g.c;
        const double rho_g = rho_i * exp(x);
        f.v[0][dst] = (real)(rp * exp(x) + g.rho_ref * expm1(x));
#pragma unroll
        for (int j = 0; j < 3; ++j) f.v[1 + j][dst] = (real)(rho_g * g.u_in[j]);
    }
}

template <typename real>
hipError_t launch_ghost(Field4<real> f, const GridDesc& gd, int axis, int bc_lo, int bc_hi, const double u_in[3],
                        double c, double rho_ref, hipStream_t s) {
    GhostArgs g;
    g.axis = axis;
    g.n = gd.n[axis];
    const int a1 = axis == 0 ? 1 : 0, a2 = axis == 2 ? 1 : 2;
    g.np1 = gd.n[a1] + 6;
    g.np2 = gd.n[a2] + 6;
    g.st_a = gd.st[axis];
    g.st_1 = gd.st[a1];
    g.st_2 = gd.st[a2];
    g.bc_lo = bc_lo;
    g.bc_hi = bc_hi;
    for (int j = 0; j < 3; ++j) g.u_in[j] = u_in[j];
    g.c = c;
    g.rho_ref = rho_ref;
    const long long total = 2LL * 3 * g.np1 * g.np2;
    const int bs = 256;
    hipLaunchKernelGGL((ghost_kernel<real>), dim3((unsigned)((total + bs - 1) / bs)), dim3(bs), 0, s, f, g);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// max |U|^2 over the interior cells (as a double; max is order independent, so the result is
// deterministic)
// ------------------------------------------------------------------------------------------------
template <typename real>
__global__ void __launch_bounds__(256) umax_kernel(Field4<real> f, GridDesc g, double rho_ref, double* part) {
    // per-workgroup maximum of |U|^2 over the interior cells; dt_kernel reduces the partial maxima
    __shared__ double red[256];
    const unsigned n = (unsigned)g.n[0] * (unsigned)g.n[1] * (unsigned)g.n[2];
    const unsigned nx = (unsigned)g.n[0], ny = (unsigned)g.n[1];
    double mx = 0.0;
    for (unsigned c = blockIdx.x * 256u + threadIdx.x; c < n; c += gridDim.x * 256u) {
        const unsigned i = c % nx, r = c / nx;
        const unsigned j = r % ny, k = r / ny;
        const long long p = g.pad0 + i + (long long)j * g.st[1] + (long long)k * g.st[2];
        const double rho = rho_ref + (double)f.v[0][p];
        const double u = (double)f.v[1][p] / rho, v = (double)f.v[2][p] / rho, w = (double)f.v[3][p] / rho;
        const double s2 = u * u + v * v + w * w;
        mx = s2 > mx ? s2 : mx;
    }
    red[threadIdx.x] = mx;
    __syncthreads();
    for (int st = 128; st > 0; st >>= 1) {
        if (threadIdx.x < st) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + st]);
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

// One launch for the ghost cells of all three axes and the [x][z][y] copy of the padded field.
// A ghost cell takes the value the axis-by-axis fill (x, then y, then z, over the full padded extent
// of the other axes) leaves there: the interior source cell is found per axis, then the boundary
// transforms of the ghost axes are applied in the order x, y, z, with the same arithmetic and the same
// rounding to the field's precision after each transform.
struct GhostAll {
    int n[3];
    int bc_lo[3], bc_hi[3];
    double u_in[3];
    double c, rho_ref;
};

// interior source index along one axis and the transform to apply (-1: none, else side 0 / 1)
__device__ __forceinline__ int ghost_source(int i, int n, int lo, int hi, int& side) {
    if (i >= 0 && i < n) {
        side = -1;
        return i;
    }
    side = i < 0 ? 0 : 1;
    const int kind = side == 0 ? lo : hi;
    if (kind == GKS_BC_PERIODIC) return side == 0 ? n + i : i - n;
    if (kind == GKS_BC_NOSLIP_WALL || kind == GKS_BC_SLIP_WALL) return side == 0 ? -1 - i : 2 * n - 1 - i;
    return side == 0 ? 0 : n - 1;  // inflow, outflow: the adjacent interior cell
}

template <typename real>
__device__ __forceinline__ void ghost_transform(real v[4], int axis, int side, int kind, const GhostAll& G) {
    if (kind == GKS_BC_NOSLIP_WALL) {
        for (int j = 1; j < 4; ++j) v[j] = -v[j];
    } else if (kind == GKS_BC_SLIP_WALL) {
        v[1 + axis] = -v[1 + axis];
    } else if (kind == GKS_BC_INFLOW) {
        const double rp = (double)v[0];
        const double rho_i = G.rho_ref + rp;
        const double un = (double)v[1 + axis] / rho_i;
        const double x = side == 0 ? (G.u_in[axis] - un) / G.c : (un - G.u_in[axis]) / G.c;
        const double rho_g = rho_i * exp(x);
        v[0] = (real)(rp * exp(x) + G.rho_ref * expm1(x));
        for (int j = 0; j < 3; ++j) v[1 + j] = (real)(rho_g * G.u_in[j]);
    }
}

// part (when not null): each workgroup's maximum of |U|^2 over its interior cells, for the CFL time step (a
// pass of its own over the field took 8.5 us on the 192 x 96 x 96 channel, 66 us on 384 x 192 x 192).
//
// Tiles of 32 x 32 cells, two cells a thread: on small grids a tile's chain of loads, boundary transforms and
// stores is what the launch takes (32^3 boxes: 256 threads of four cells each made the FP32 step 3.1 us and the
// FP64 step 2.7 us longer, 48.1 and 78.0 us; 1024 threads gain 0.4 us there and lose 0.9 % on 192 x 96 x 96). On
// large grids it is bound by memory, 32 B (FP32) or 64 B a cell, and by the lines that rows of X and Y cells share
// at their ends: x runs fastest and neighbouring workgroups go to one XCD, so that both parts of such a line
// meet in its L2 (z fastest: 384 x 192 x 192 FP32 0.7 %, 192 x 96 x 96 1.1 % of the step). Tiles of 64 x 64 are no
// faster there (0.3 %, and 4 % slower on 32^3), tiles of 16 rows 2 % slower.
constexpr int GHOST_TILE = 32, GHOST_THREADS = 512;

//
// RESTORE: a step's state for its adjoint. The interior is read from a checkpoint (`from`) and every cell written to
// q; the launch before stage 2 sets the step's time (t). The adjoint's x direction reads the copy. Bound by
// memory: 56 us on 128^3, 7.2 us on 48^3 for 32 B a cell read and 64 B written.
template <typename real, bool RESTORE>
__global__ void __launch_bounds__(GHOST_THREADS) ghost_transpose_kernel(Field4<const real> from, Field4<real> q,
                                                                        Field4<real> qt, GhostAll G, double* part,
                                                                        int n_wg, const double* t_n, const DtArgs dt) {
    constexpr int T = GHOST_TILE, RS = GHOST_THREADS / T, NR = T / RS;
    __shared__ real t[4][T][T + 1];
    __shared__ double s_max[GHOST_THREADS / 64];
    double mx = 0.0;
    const int X = G.n[0] + 6, Y = G.n[1] + 6, Z = G.n[2] + 6;
    const int tx = threadIdx.x % T, ty = threadIdx.x / T;
    const int blk = (blockIdx.x % 8) * (gridDim.x / 8) + blockIdx.x / 8;
    if (blk >= n_wg) return;
    const int nx = (X + T - 1) / T;
    const int x0 = blk % nx * T, z = blk / nx % Z, y0 = blk / nx / Z * T;
    // every lane finds the cell its value comes from (itself inside the domain, the interior source of
    // a ghost cell) and all its loads are issued before any is used; cells outside the padded block read
    // cell 0 and are not used
    int sd[NR][3];
    long long src[NR], dst[NR];
    bool in[NR], gh[NR];
    const int sk = ghost_source(z - 3, G.n[2], G.bc_lo[2], G.bc_hi[2], sd[0][2]);
#pragma unroll
    for (int i = 0; i < NR; ++i) {
        const int x = x0 + tx, y = y0 + ty + RS * i;
        in[i] = x < X && y < Y;
        sd[i][2] = sd[0][2];
        const int si = ghost_source(x - 3, G.n[0], G.bc_lo[0], G.bc_hi[0], sd[i][0]);
        const int sj = ghost_source(y - 3, G.n[1], G.bc_lo[1], G.bc_hi[1], sd[i][1]);
        gh[i] = in[i] && (sd[i][0] >= 0 || sd[i][1] >= 0 || sd[i][2] >= 0);
        dst[i] = ((long long)z * Y + y) * X + x;
        src[i] = in[i] ? ((long long)(sk + 3) * Y + (sj + 3)) * X + (si + 3) : 0;
    }
    real v[NR][4];
#pragma unroll
    for (int i = 0; i < NR; ++i)
#pragma unroll
        for (int w = 0; w < 4; ++w) v[i][w] = from.v[w][src[i]];
#pragma unroll
    for (int i = 0; i < NR; ++i) {
        if (gh[i]) {
            for (int a = 0; a < 3; ++a)
                if (sd[i][a] >= 0) ghost_transform(v[i], a, sd[i][a], sd[i][a] == 0 ? G.bc_lo[a] : G.bc_hi[a], G);
        }
        if (RESTORE ? in[i] : gh[i])
#pragma unroll
            for (int w = 0; w < 4; ++w) q.v[w][dst[i]] = v[i][w];
#pragma unroll
        for (int w = 0; w < 4; ++w) t[w][ty + RS * i][tx] = v[i][w];
        if (part && in[i] && !gh[i]) {
            const double rho = G.rho_ref + (double)v[i][0];
            const double mx_ = (double)v[i][1], my_ = (double)v[i][2], mz_ = (double)v[i][3];
            const double s2 = (mx_ * mx_ + my_ * my_ + mz_ * mz_) / (rho * rho);
            mx = s2 > mx ? s2 : mx;
        }
    }
    if (part) {
        for (int o = 32; o > 0; o >>= 1) mx = fmax(mx, __shfl_xor(mx, o));
        if ((threadIdx.x & 63) == 0) s_max[threadIdx.x >> 6] = mx;
    }
    __syncthreads();
    if (part && threadIdx.x == 0) {
        for (int w = 1; w < GHOST_THREADS / 64; ++w) mx = fmax(mx, s_max[w]);
        part[blk] = mx;
    }
#pragma unroll
    for (int w = 0; w < 4; ++w)
#pragma unroll
        for (int r = ty; r < T; r += RS) {
            const int y = y0 + tx, x = x0 + r;
            if (x < X && y < Y) qt.v[w][((long long)x * Z + z) * Y + y] = t[w][tx][r];
        }
    if (RESTORE && t_n && blk == 0) {
        if (threadIdx.x == 0) dt.st->t = *t_n;
        dt_update<GHOST_THREADS>(dt, s_max);
    }
}

GhostAll ghost_args(const GridDesc& gd, const int bc[6], const double u_in[3], double c, double rho_ref) {
    GhostAll G;
    for (int a = 0; a < 3; ++a) {
        G.n[a] = gd.n[a];
        G.bc_lo[a] = bc[2 * a];
        G.bc_hi[a] = bc[2 * a + 1];
        G.u_in[a] = u_in[a];
    }
    G.c = c;
    G.rho_ref = rho_ref;
    return G;
}

// the value of cell (x, y, z), 0 .. n - 1 inside the domain, ghost cells filled from the interior of q
template <typename real, typename Field>
__device__ __forceinline__ void ghost_value(const Field& q, int x, int y, int z, const GhostAll& G, real v[4]) {
    int sd[3];
    const int si = ghost_source(x, G.n[0], G.bc_lo[0], G.bc_hi[0], sd[0]);
    const int sj = ghost_source(y, G.n[1], G.bc_lo[1], G.bc_hi[1], sd[1]);
    const int sk = ghost_source(z, G.n[2], G.bc_lo[2], G.bc_hi[2], sd[2]);
    const long long src = ((long long)(sk + 3) * (G.n[1] + 6) + (sj + 3)) * (G.n[0] + 6) + (si + 3);
#pragma unroll
    for (int w = 0; w < 4; ++w) v[w] = q.v[w][src];
    for (int a = 0; a < 3; ++a)
        if (sd[a] >= 0) ghost_transform(v, a, sd[a], sd[a] == 0 ? G.bc_lo[a] : G.bc_hi[a], G);
}

// The ghost cells alone, one thread each, for passes that need no copy of the field: the six z planes, then
// the y rows of the interior planes, then the x ends of the interior rows.
template <typename real>
__global__ void __launch_bounds__(256) ghost_shell_kernel(Field4<real> q, GhostAll G) {
    const int X = G.n[0] + 6, Y = G.n[1] + 6;
    const long long nz = 6LL * X * Y, ny = 6LL * X * G.n[2], nx = 6LL * G.n[1] * G.n[2];
    long long t = (long long)blockIdx.x * 256 + threadIdx.x;
    int x, y, z;
    auto ghost = [](int s, int n) { return s < 3 ? s - 3 : n + s - 3; };
    if (t < nz) {
        x = (int)(t % X) - 3;
        y = (int)(t / X % Y) - 3;
        z = ghost((int)(t / ((long long)X * Y)), G.n[2]);
    } else if ((t -= nz) < ny) {
        x = (int)(t % X) - 3;
        y = ghost((int)(t / X % 6), G.n[1]);
        z = (int)(t / (6LL * X));
    } else if ((t -= ny) < nx) {
        x = ghost((int)(t % 6), G.n[0]);
        y = (int)(t / 6 % G.n[1]);
        z = (int)(t / (6LL * G.n[1]));
    } else {
        return;
    }
    real v[4];
    ghost_value(q, x, y, z, G, v);
    const long long dst = ((long long)(z + 3) * Y + (y + 3)) * X + (x + 3);
#pragma unroll
    for (int w = 0; w < 4; ++w) q.v[w][dst] = v[w];
}

template <typename real>
hipError_t launch_ghost_shell(Field4<real> q, const GridDesc& gd, const int bc[6], const double u_in[3], double c,
                              double rho_ref, hipStream_t s) {
    const GhostAll G = ghost_args(gd, bc, u_in, c, rho_ref);
    const long long X = gd.n[0] + 6, Y = gd.n[1] + 6;
    const long long total = 6 * (X * Y + X * gd.n[2] + (long long)gd.n[1] * gd.n[2]);
    hipLaunchKernelGGL((ghost_shell_kernel<real>), dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, q, G);
    return hipGetLastError();
}

template <typename real>
hipError_t launch_ghost_transpose(Field4<real> q, Field4<real> qt, const GridDesc& gd, const int bc[6],
                                  const double u_in[3], double c, double rho_ref, double* part, hipStream_t s) {
    const GhostAll G = ghost_args(gd, bc, u_in, c, rho_ref);
    const int n_wg = ghost_parts(gd.n);
    Field4<const real> from;
    for (int v = 0; v < 4; ++v) from.v[v] = q.v[v];
    hipLaunchKernelGGL((ghost_transpose_kernel<real, false>), dim3(pad8(n_wg)), dim3(GHOST_THREADS), 0, s, from, q, qt, G,
                       part, n_wg, nullptr, DtArgs{});
    return hipGetLastError();
}

hipError_t launch_restore(const double* const from[4], Field4<double> q, Field4<double> qt, const GridDesc& gd,
                          const int bc[6], const double u_in[3], double c, double rho_ref, const double* t,
                          const DtArgs& dt, hipStream_t s) {
    Field4<const double> f;
    for (int v = 0; v < 4; ++v) f.v[v] = from[v];
    const int n_wg = ghost_parts(gd.n);
    hipLaunchKernelGGL((ghost_transpose_kernel<double, true>), dim3(pad8(n_wg)), dim3(GHOST_THREADS), 0, s, f, q, qt,
                       ghost_args(gd, bc, u_in, c, rho_ref), nullptr, n_wg, t, dt);
    return hipGetLastError();
}

// Stage update from the three directions' residuals, for launches in which they run side by side: one thread
// per cell. The z pass's residual stands in the output fields; it and the sums are formed as in the z pass.
// Bound by memory: FP32 192 B a cell in stage 1 and 112 B in stage 2.
template <typename real>
struct Vec4T;
template <>
struct Vec4T<float> {
    using type = float4;
};
template <>
struct Vec4T<double> {
    using type = double4;
};
template <typename real>
__device__ __forceinline__ void load4(const real* p, long long i, real v[4]) {
    const typename Vec4T<real>::type x = *reinterpret_cast<const typename Vec4T<real>::type*>(p + 4 * i);
    v[0] = x.x, v[1] = x.y, v[2] = x.z, v[3] = x.w;
}
template <typename real>
__device__ __forceinline__ void store4(real* p, long long i, const real v[4]) {
    typename Vec4T<real>::type x;
    x.x = v[0], x.y = v[1], x.z = v[2], x.w = v[3];
    *reinterpret_cast<typename Vec4T<real>::type*>(p + 4 * i) = x;
}

template <typename real, int STAGE>
__global__ void __launch_bounds__(256) combine_kernel(const FaceArgs<real> a, GridDesc g) {
    constexpr bool F0 = STAGE == 1, COMP = sizeof(real) == 4;
    constexpr int LOC[4] = {LocalOrder<5>::v[0], LocalOrder<5>::v[1], LocalOrder<5>::v[2], LocalOrder<5>::v[3]};
    const long long n = (long long)g.n[0] * g.n[1] * g.n[2];
    const long long c = (long long)blockIdx.x * 256 + threadIdx.x;
    if (a.finish && c == 0) finish_step(a.finish);
    if (c >= n) return;
    const int i = (int)(c % g.n[0]);
    const long long r = c / g.n[0];
    const int j = (int)(r % g.n[1]), k = (int)(r / g.n[1]);
    const long long p = g.pad0 + i + (long long)j * g.st[1] + (long long)k * g.st[2];
    const long long x = rx_block_index(i, j, k, a.rx_nx, a.rx_nyb);
    const real dt = real(*a.dt_ptr);
    real r1[4], x1[4], r0[4] = {}, x0[4] = {}, lo[4] = {}, la[4] = {}, lb[4] = {};
    load4(a.r1, c, r1);
    load4(a.rx1, x, x1);
    if (F0) {
        load4(a.r0, c, r0);
        load4(a.rx0, x, x0);
    }
    if (COMP) load4(a.lo_in, c, lo);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        real* const oa = a.out_a[LOC[v]];
        real* const ob = a.out_b[LOC[v]];
        const real L1 = r1[v] + (oa[p] + x1[v]);
        const real L0 = F0 ? r0[v] + (ob[p] + x0[v]) : real(0);
        const real q = F0 ? a.q_c[LOC[v]][p] : a.s_in[LOC[v]][p];
        const real add = F0 ? real(0.5) * dt * L0 + real(0.125) * dt * dt * L1
                            : (dt * dt * real(1.0 / 3.0)) * L1 + (v > 0 ? dt * a.g_global[v > 0 ? v - 1 : 0] : real(0));
        const real add2 = F0 ? dt * L0 + (dt * dt * real(1.0 / 6.0)) * L1 : real(0);
        if constexpr (COMP) {
            float sh, sl;
            two_sum(q, lo[v] + add, sh, sl);
            oa[p] = sh;
            la[v] = sl;
            if (F0) {
                two_sum(q, lo[v] + add2, sh, sl);
                ob[p] = sh;
                lb[v] = sl;
            }
        } else {
            oa[p] = q + add;
            if (F0) ob[p] = q + add2;
        }
    }
    if constexpr (COMP) {
        store4(a.lo_a, c, la);
        if (F0) store4(a.lo_b, c, lb);
    }
}

template <typename real>
hipError_t launch_combine(const FaceArgs<real>& az, const GridDesc& g, int stage, hipStream_t s) {
    const long long n = (long long)g.n[0] * g.n[1] * g.n[2];
    const dim3 grid((unsigned)((n + 255) / 256)), block(256);
    if (stage == 1) hipLaunchKernelGGL((combine_kernel<real, 1>), grid, block, 0, s, az, g);
    else hipLaunchKernelGGL((combine_kernel<real, 2>), grid, block, 0, s, az, g);
    return hipGetLastError();
}

int umax_parts(const int n[3]) { return (int)std::min(((long long)n[0] * n[1] * n[2] + 255) / 256, (long long)UMAX_BLOCKS); }
// workgroups of the ghost fill
int ghost_parts(const int n[3]) {
    constexpr int T = GHOST_TILE;
    return (n[2] + 6) * ((n[0] + 6 + T - 1) / T) * ((n[1] + 6 + T - 1) / T);
}

template <typename real>
hipError_t launch_umax(Field4<real> f, const GridDesc& g, double rho_ref, double* part, hipStream_t s) {
    hipLaunchKernelGGL((umax_kernel<real>), dim3((unsigned)umax_parts(g.n)), dim3(256), 0, s, f, g, rho_ref, part);
    return hipGetLastError();
}

__global__ void __launch_bounds__(DT_THREADS) dt_kernel(const DtArgs a) {
    __shared__ double red[DT_THREADS / 64];
    dt_update<DT_THREADS>(a, red);
}

hipError_t launch_dt(const DtArgs& a, hipStream_t s) {
    hipLaunchKernelGGL(dt_kernel, dim3(1), dim3(DT_THREADS), 0, s, a);
    return hipGetLastError();
}

__global__ void finish_kernel(DevState* st, int has_rotor, double* hist) {
    if (threadIdx.x != 0) return;
    finish_step(st);
    if (has_rotor) {
        st->win_p += st->power;
        st->win_t += st->thrust;
    }
    if (hist) {
        double h[10];
        h[0] = st->t;
        h[1] = st->dt;
        h[2] = st->thrust;
        h[3] = st->torque;
        h[4] = st->power;
        h[5] = st->cp;
        h[6] = st->ct;
        h[7] = st->ibm_force[0];
        h[8] = st->ibm_force[1];
        h[9] = st->ibm_force[2];
        for (int i = 0; i < 10; ++i) hist[i] = h[i];
    }
}

hipError_t launch_finish(DevState* st, int has_rotor, double* hist, hipStream_t s) {
    hipLaunchKernelGGL(finish_kernel, dim3(1), dim3(64), 0, s, st, has_rotor, hist);
    return hipGetLastError();
}

__global__ void window_reset_kernel(DevState* st) {
    if (threadIdx.x != 0) return;
    st->win_p = 0.0;
    st->win_t = 0.0;
    st->win_n = 0;
}

hipError_t launch_window_reset(DevState* st, hipStream_t s) {
    hipLaunchKernelGGL(window_reset_kernel, dim3(1), dim3(64), 0, s, st);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// FP64 conservation sums, max |U| and a non-finite flag; fixed-order block partials then one block
// ------------------------------------------------------------------------------------------------
int diag_blocks(const GridDesc& g) {
    const long long n = (long long)g.n[0] * g.n[1] * g.n[2];
    long long b = (n + 255) / 256;
    if (b > 1024) b = 1024;
    return (int)b;
}

template <typename real>
__global__ void __launch_bounds__(256) diag_kernel(Field4<real> f, const real* lo, GridDesc g, double rho_ref,
                                                   double* partials, DevState* st) {
    __shared__ double red[4][256];
    __shared__ double mxs[256];
    const long long n = (long long)g.n[0] * g.n[1] * g.n[2];
    double s[4] = {0, 0, 0, 0};
    double mx = 0.0;
    int bad = 0;
    for (long long c = (long long)blockIdx.x * blockDim.x + threadIdx.x; c < n; c += (long long)gridDim.x * blockDim.x) {
        const int i = (int)(c % g.n[0]);
        const long long r = c / g.n[0];
        const int j = (int)(r % g.n[1]);
        const int k = (int)(r / g.n[1]);
        const long long p = g.pad0 + i * g.st[0] + j * g.st[1] + (long long)k * g.st[2];
        double q[4];
        // stretched axes: each cell weighs its volume over the mean cell volume (exactly 1 when uniform)
        const double wgt = (g.wrel[0] ? g.wrel[0][i] : 1.0) * (g.wrel[1] ? g.wrel[1][j] : 1.0) *
                           (g.wrel[2] ? g.wrel[2][k] : 1.0);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            // FP32: the state is the field plus its low-order part ([cell][4], interior cells)
            q[v] = lo ? (double)f.v[v][p] + (double)lo[4 * c + v] : (double)f.v[v][p];
            s[v] += q[v] * wgt;
            if (!isfinite(q[v])) bad = 1;
        }
        const double rho = rho_ref + q[0];
        const double s2 = (q[1] * q[1] + q[2] * q[2] + q[3] * q[3]) / (rho * rho);
        mx = s2 > mx ? s2 : mx;
    }
    for (int v = 0; v < 4; ++v) red[v][threadIdx.x] = s[v];
    mxs[threadIdx.x] = mx;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < w) {
            for (int v = 0; v < 4; ++v) red[v][threadIdx.x] += red[v][threadIdx.x + w];
            mxs[threadIdx.x] = fmax(mxs[threadIdx.x], mxs[threadIdx.x + w]);
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        for (int v = 0; v < 4; ++v) partials[4 * blockIdx.x + v] = red[v][0];
        atomicMax(&st->umax_diag_bits, (unsigned long long)__double_as_longlong(mxs[0]));
    }
    if (bad) atomicOr(&st->nonfinite, 1);
}

__global__ void __launch_bounds__(256) diag_final_kernel(const double* partials, int nblk, DevState* st, double vol) {
    __shared__ double red[4][256];
    double s[4] = {0, 0, 0, 0};
    for (int b = threadIdx.x; b < nblk; b += blockDim.x)
        for (int v = 0; v < 4; ++v) s[v] += partials[4 * b + v];
    for (int v = 0; v < 4; ++v) red[v][threadIdx.x] = s[v];
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < w)
            for (int v = 0; v < 4; ++v) red[v][threadIdx.x] += red[v][threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        st->mass = red[0][0] * vol;
        for (int v = 0; v < 3; ++v) st->mom[v] = red[1 + v][0] * vol;
    }
}

__global__ void diag_reset_kernel(DevState* st) {
    if (threadIdx.x == 0) {
        st->umax_diag_bits = 0ULL;
        st->nonfinite = 0;
    }
}

template <typename real>
hipError_t launch_diag(Field4<real> f, const real* lo, const GridDesc& g, double rho_ref, double* partials, int nblk,
                       DevState* st, hipStream_t s) {
    hipLaunchKernelGGL(diag_reset_kernel, dim3(1), dim3(64), 0, s, st);
    hipLaunchKernelGGL((diag_kernel<real>), dim3(nblk), dim3(256), 0, s, f, lo, g, rho_ref, partials, st);
    hipLaunchKernelGGL(diag_final_kernel, dim3(1), dim3(256), 0, s, (const double*)partials, nblk, st,
                       g.h[0] * g.h[1] * g.h[2]);
    return hipGetLastError();
}

// zero-fill of device memory by a kernel (usable inside a captured graph, unlike a memset node)
__global__ void __launch_bounds__(256) zero_words_kernel(unsigned* p, long long n) {
    for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < n; i += (long long)gridDim.x * 256) p[i] = 0u;
}

hipError_t launch_zero_words(void* p, size_t bytes, hipStream_t s) {
    const long long n = (long long)(bytes / 4);
    if (n <= 0) return hipSuccess;
    long long blocks = (n + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(zero_words_kernel, dim3((unsigned)blocks), dim3(256), 0, s, static_cast<unsigned*>(p), n);
    return hipGetLastError();
}

hipError_t launch_copy_field(const void* src, void* dst, size_t bytes, hipStream_t s) {
    return hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToDevice, s);
}

template hipError_t launch_ghost<float>(Field4<float>, const GridDesc&, int, int, int, const double*, double, double, hipStream_t);
template hipError_t launch_ghost<double>(Field4<double>, const GridDesc&, int, int, int, const double*, double, double, hipStream_t);
template hipError_t launch_ghost_transpose<float>(Field4<float>, Field4<float>, const GridDesc&, const int[6], const double[3], double, double, double*, hipStream_t);
template hipError_t launch_ghost_transpose<double>(Field4<double>, Field4<double>, const GridDesc&, const int[6], const double[3], double, double, double*, hipStream_t);
template hipError_t launch_ghost_shell<float>(Field4<float>, const GridDesc&, const int[6], const double[3], double, double, hipStream_t);
template hipError_t launch_ghost_shell<double>(Field4<double>, const GridDesc&, const int[6], const double[3], double, double, hipStream_t);
template hipError_t launch_combine<float>(const FaceArgs<float>&, const GridDesc&, int, hipStream_t);
template hipError_t launch_combine<double>(const FaceArgs<double>&, const GridDesc&, int, hipStream_t);
template hipError_t launch_umax<float>(Field4<float>, const GridDesc&, double, double*, hipStream_t);
template hipError_t launch_umax<double>(Field4<double>, const GridDesc&, double, double*, hipStream_t);
template hipError_t launch_diag<float>(Field4<float>, const float*, const GridDesc&, double, double*, int, DevState*,
                                      hipStream_t);
template hipError_t launch_diag<double>(Field4<double>, const double*, const GridDesc&, double, double*, int,
                                       DevState*, hipStream_t);

}  // namespace gks
