// gks_stage64.hip -- the FP64 S2O4 stage kernels (the FP32 ones are in gks_stage.hip): reconstruction,
// gas-kinetic flux, flux divergence and the stage combination, the x and y directions in one launch and z in one,
// or all three together on small grids (Section 2, Eqs. (semi), (finite), (x_example), (flux); the two-stage
// fourth-order combinations).
//
// One workgroup owns a tile of 16 x T2 faces in the tangential plane and marches along the normal over its
// share of the tile-major (tile, cell) order (face_split). FOUR lanes work on a face: lane bits 2 (h) and 3
// (m). What bounds the kernel is FP64 vector issue and the dependent-instruction latency behind it, so it
// needs several waves per SIMD, and the state of a whole face line (40 doubles of Gauss-point values, a
// 28-double column window) does not fit their registers: with two lanes per face, one wave per SIMD, 28 % of
// the instructions moved values to and from the accumulation registers. The split halves both:
//   * column phase: a thread owns one tangential column of the tile and its two-cell halo and TWO of the four
//     variables (waves of the lower half take density and normal momentum, the others the tangential momenta);
//     it keeps a five-cell window and writes the WENO-JS values of both faces, the normal derivative D and
//     C = (q^L + q^R)/2 to LDS;
//   * t1 phase: a wave takes a row of all four variables, 16 positions each: WENO-JS at the two Gauss points
//     of q^L, q^R, quartic values of D and C and the quartic derivative of C -> LDS;
//   * t2 phase: lane (h, m) evaluates Gauss line m for variables 2h, 2h + 1 at both Gauss points of the line;
//   * the lanes of a pair (m fixed) exchange through DPP so that lane h holds all four variables at Gauss
//     point h, and each evaluates one flux;
//   * a reduce-scatter over the four lanes leaves lane (h, m) the face flux of global variable 2h + m, whose
//     divergence, accumulation or stage update it does.
// Measured, 192 x 96 x 96 channel: 1.85 ms a step with two lanes per face, 1.56 ms with four (12-row tiles, three
// waves per SIMD), 1.45 ms with the directions sharing launches, 1.39 ms with the LDS layout below; the tile height is
// chosen per grid, one for all directions (FACE64_ROWS, face_plan).
#include "gks_internal.h"

namespace gks {

namespace {

template <typename T>
__device__ __forceinline__ T sel(bool c, T x, T y) {
    return c ? x : y;
}

}  // namespace

// LDS, per variable: column values [q^L, q^R, D, C][t2 row][t1 column] and t1-phase results
// [q^L_m, q^R_m, D_m, (dC/dt1)_m, C_m][t2 row][Gauss line m][t1 position]. A 64-bit access takes 16 lanes at a time
// over 32 banks: the t1 phase reads and stores 16 positions of one variable and line; the t2 phase reads four
// faces of both lines of the variables v and v + 2, so lines start 8 words apart modulo 32 and those variables'
// blocks 16. (With the lines interleaved, 128-bit stores, and the blocks 32 words apart: 55 M conflict cycles in a
// stage-1 x and y launch of the 192 x 96 x 96 channel, now 4.5 M; 1.43 ms a step, now 1.39; 32^3 75.1 us, now 71.4.)
template <int X2>
struct Face64Lds {
    struct {
        double a[4][X2][EXT1];
        double pad[(16 - (4 * X2 * EXT1) % 32 + 32) % 32];
    } nrm[4];
    struct {
        double a[5][X2][2][TILE1 + 4];
        double pad[(4 - (5 * X2 * 2 * (TILE1 + 4)) % 32 + 32) % 32];
    } t1[4];
};

// The marches of workgroup blk of the nblk (a multiple of 8) that take this direction.
// MODE (the direction's role): 3 = x pass, writes its residual to the blocked arrays; 0 = y pass,
// writes the main residual arrays; 4 = z pass, adds both and applies the S2O4 stage update; 5 = z pass
// beside the other two, leaves its residual where the stage update will stand (combine_kernel does it).
// STR: the mesh is stretched and the spacings come from the per-axis arrays; otherwise the uniform
// inverse spacings are kernel arguments. T2: rows of the tile; a wave per row.
template <int T2, int STAGE, int MODE, bool STR>
__device__ __forceinline__ void face64_march(const FaceArgs<double>& a, const int blk, const int nblk,
                                             Face64Lds<T2 + 4>& lds) {
    static_assert(MODE == 0 || MODE == 3 || MODE == 4 || MODE == 5, "face pass mode");
    constexpr int X2 = T2 + 4, NTH = 64 * T2;
    static_assert(TILE1 == 16 && NTH == 4 * TILE1 * T2 && 2 * EXT1 * X2 <= NTH,
                  "four lanes per face, a wave per t2 row, two threads per column");
    constexpr bool NEED_F0 = (STAGE == 1);
    constexpr int LOC[4] = {LocalOrder<MODE>::v[0], LocalOrder<MODE>::v[1], LocalOrder<MODE>::v[2],
                            LocalOrder<MODE>::v[3]};
    auto& s_nrm = lds.nrm;
    auto& s_t1 = lds.t1;

    const int tid = threadIdx.x;
    // consecutive logical workgroups run on the same XCD (the hardware deals workgroups round-robin to
    // the 8 XCDs; the grid is padded to a multiple of 8), so neighbouring tiles share that XCD's L2 for
    // their halo columns
    const int b = (blk % 8) * (nblk / 8) + blk / 8;
    if (b >= a.n_wg) return;
    // this workgroup's cells as a range [lin, lin_end) of the tile-major (tile, cell) order
    const int tiles = a.tiles_t1 * a.tiles_t2;
    long long lin, lin_end;
    if (a.seg_len > 0) {
        lin = (long long)b * a.seg_len;
        lin_end = min(lin + a.seg_len, (long long)tiles * a.n_n);
    } else {
        const int c0 = (b / tiles) * a.chunk;
        lin = (long long)(b % tiles) * a.n_n + c0;
        lin_end = lin + min(a.chunk, a.n_n - c0);
    }

    // column role: variables cv, cv + 1 of column (c1, c2); cv is uniform over a wave
    const int half = __builtin_amdgcn_readfirstlane(tid / (NTH / 2));
    const int cv = 2 * half, ct = tid % (NTH / 2);
    const bool col = ct < EXT1 * X2;
    const int c1 = ct % EXT1, c2 = ct / EXT1;
    const double* const qcol[2] = {half ? a.q[2] : a.q[0], half ? a.q[3] : a.q[1]};
    // face role: face (fj, fk), variable pair / Gauss point h, Gauss line m
    const int hi = (tid >> 2) & 1, m = (tid >> 3) & 1;
    const bool h = hi != 0, mb = m != 0;
    const int fj = (tid & 3) + 4 * ((tid >> 4) & 3), fk = tid >> 6;
    const int gvar = 2 * hi + m;  // global variable whose flux this lane ends up with
    // this lane's fields and body force in the z pass
    auto lane_field = [&](auto* const(&p)[4]) {
        return sel(h, sel(mb, p[LOC[3]], p[LOC[2]]), sel(mb, p[LOC[1]], p[LOC[0]]));
    };
    const double* const src = NEED_F0 ? lane_field(a.q_c) : lane_field(a.s_in);
    double* const out_a = lane_field(a.out_a);
    double* const out_b = lane_field(a.out_b);
    const double gforce = sel(h, sel(mb, a.g_global[2], a.g_global[1]), sel(mb, a.g_global[0], 0.0));
    const double dt = *a.dt_ptr;
    const double eps = a.eps;

    // one march per tile the range meets (the window and the face fluxes restart)
    while (lin < lin_end) {
        const int tile = (int)(lin / a.n_n);
        const int f0 = (int)(lin - (long long)tile * a.n_n);
        const int f1 = (int)min((long long)a.n_n, f0 + (lin_end - lin));  // residuals of cells [f0, f1); faces f0..f1
        lin += f1 - f0;
        const int tile1 = tile % a.tiles_t1, tile2 = tile / a.tiles_t1;
        const int j0 = tile1 * TILE1, k0 = tile2 * T2;
        // columns outside the padded domain and threads without a column read a clamped column, whose
        // values reach no face of the domain
        const int jc = min(j0 - 2 + c1, a.n_t1 + NG - 1), kc = min(k0 - 2 + min(c2, X2 - 1), a.n_t2 + NG - 1);
        const long long cbase = a.pad0 + (long long)jc * a.st_t1 + (long long)kc * a.st_t2;
        const bool face_ok = (j0 + fj < a.n_t1) && (k0 + fk < a.n_t2);
        const int je = min(j0 + fj, a.n_t1 - 1), ke = min(k0 + fk, a.n_t2 - 1);
        const long long rbase = (long long)je * a.ist_t1 + (long long)ke * a.ist_t2;
        const long long pbase = a.pad0 + (long long)je * a.st_t1 + (long long)ke * a.st_t2;
        const double ih2 = STR ? a.ih2[ke] : a.inv_h2;
        const double ih1 = STR ? a.ih1[min(j0 + (tid & 15), a.n_t1 - 1)] : a.inv_h1;

        // window of cells f0-3 .. f0+1, the right-face value of cell f0-1 (q^L of face f0) and the cell that
        // enters at the first step (each next cell is loaded one step ahead)
        double ring[2][5], carry[2], nxt[2];
#pragma unroll
        for (int v = 0; v < 2; ++v) {
#pragma unroll
            for (int r = 0; r < 5; ++r) ring[v][r] = qcol[v][cbase + (long long)(f0 - 3 + r) * a.st_n];
            nxt[v] = qcol[v][cbase + (long long)(f0 + 2) * a.st_n];
        }
#pragma unroll
        for (int v = 0; v < 2; ++v) {
            double left;
            weno_faces<double>(ring[v][0], ring[v][1], ring[v][2], ring[v][3], ring[v][4], eps, carry[v], left);
        }
        double prev0 = 0.0, prev1 = 0.0;  // this lane's fluxes of the previous face

        for (int f = f0; f <= f1; ++f) {
            // epilogue operands of cell f - 1 (z pass), loaded a step's arithmetic ahead; at f = f0 and for
            // faces outside the domain a clamped cell is read and its values are not used
            const int ce = max(f - 1, 0);
            const long long ridx = 4 * (rbase + (long long)ce * a.ist_n) + gvar;
            const long long pidx = pbase + (long long)ce * a.st_n;
            double r0v = 0.0, r1v = 0.0, x0v = 0.0, x1v = 0.0, qe = 0.0;
            if constexpr (MODE == 4) {
                const long long xidx = 4 * rx_block_index(je, ke, ce, a.rx_nx, a.rx_nyb) + gvar;
                r1v = a.r1[ridx];
                x1v = a.rx1[xidx];
                if (NEED_F0) {
                    r0v = a.r0[ridx];
                    x0v = a.rx0[xidx];
                }
                qe = src[pidx];
            }
            // ---- column phase: window cells f-2 .. f+2, prefetch cell f+3
            {
                const double ihf_f = STR ? a.ihf[f] : a.inv_hn;
                const long long idx = cbase + (long long)min(f + 3, a.n_n + 2) * a.st_n;
#pragma unroll
                for (int v = 0; v < 2; ++v) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) ring[v][r] = ring[v][r + 1];
                    ring[v][4] = nxt[v];
                    nxt[v] = qcol[v][idx];
                }
                if (col) {
#pragma unroll
                    for (int v = 0; v < 2; ++v) {
                        double right, left;
                        weno_faces<double>(ring[v][0], ring[v][1], ring[v][2], ring[v][3], ring[v][4], eps, right, left);
                        const double qL = carry[v];
                        s_nrm[cv + v].a[0][c2][c1] = qL;
                        s_nrm[cv + v].a[1][c2][c1] = left;
                        s_nrm[cv + v].a[2][c2][c1] = (ring[v][0] - 15.0 * ring[v][1] + 15.0 * ring[v][2] - ring[v][3]) *
                                                     ((1.0 / 12.0) * ihf_f);
                        s_nrm[cv + v].a[3][c2][c1] = 0.5 * (qL + left);
                        carry[v] = right;
                    }
                }
            }
            __syncthreads();
            // ---- t1 phase: a wave takes rows tid / 64 + k T2, 16 positions of all four variables
            {
                const int tj = tid & 15, v = (tid >> 4) & 3;
#pragma unroll
                for (int kk = 0; kk < (X2 + T2 - 1) / T2; ++kk) {
                    const int tk = (tid >> 6) + kk * T2;
                    if (tk < X2) {
                        double x[5], vm, vp;
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
#pragma unroll
                            for (int r = 0; r < 5; ++r) x[r] = s_nrm[v].a[q][tk][tj + r];
                            if (q < 2) weno_gauss<double>(x[0], x[1], x[2], x[3], x[4], eps, vm, vp);
                            else quartic_gauss_value<double>(x[0], x[1], x[2], x[3], x[4], vm, vp);
                            s_t1[v].a[q == 3 ? 4 : q][tk][0][tj] = vm;
                            s_t1[v].a[q == 3 ? 4 : q][tk][1][tj] = vp;
                            if (q == 3) {
                                quartic_gauss_deriv<double>(x[0], x[1], x[2], x[3], x[4], vm, vp);
                                s_t1[v].a[3][tk][0][tj] = vm * ih1;
                                s_t1[v].a[3][tk][1][tj] = vp * ih1;
                            }
                        }
                    }
                }
            }
            __syncthreads();
            // ---- t2 phase: variables 2h, 2h + 1 of Gauss line m at its two Gauss points
            double gp[2][2][5];  // [variable][Gauss n][q^L, q^R, d/dn, d/dt1, d/dt2]
#pragma unroll
            for (int v = 0; v < 2; ++v) {
                const auto& t = s_t1[2 * hi + v];
#pragma unroll
                for (int q = 0; q < 5; ++q) {
                    double y[5];
#pragma unroll
                    for (int r = 0; r < 5; ++r) y[r] = t.a[q][fk + r][m][fj];
                    double vm, vp;
                    if (q < 2) weno_gauss<double>(y[0], y[1], y[2], y[3], y[4], eps, vm, vp);
                    else if (q < 4) quartic_gauss_value<double>(y[0], y[1], y[2], y[3], y[4], vm, vp);
                    else {
                        quartic_gauss_deriv<double>(y[0], y[1], y[2], y[3], y[4], vm, vp);
                        vm *= ih2;
                        vp *= ih2;
                    }
                    gp[v][0][q] = vm;
                    gp[v][1][q] = vp;
                }
            }
            // ---- exchange in the lane pair: all four variables at Gauss point n = h
            double w[4][5];
#pragma unroll
            for (int v = 0; v < 2; ++v)
#pragma unroll
                for (int q = 0; q < 5; ++q) {
                    w[v][q] = dpp_move<ROW_SHR4, BANK_H1>(gp[v][0][q], gp[v][1][q]);
                    w[2 + v][q] = dpp_move<ROW_SHL4, BANK_H0>(gp[v][1][q], gp[v][0][q]);
                }
            double fa0[4], fa1[4];
            {
                double qL[4], qR[4], g[3][4];
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    qL[v] = w[v][0];
                    qR[v] = w[v][1];
                    g[0][v] = w[v][2];
                    g[1][v] = w[v][3];
                    g[2][v] = w[v][4];
                }
                gp_flux<double, NEED_F0>(qL, qR, g, a.fc, fa0, fa1);
            }
            // ---- sum over the four Gauss points, scattered: lane (h, m) keeps global variable 2h + m
            auto scatter_sum = [&](const double(&x)[4]) {
                double y[2];
#pragma unroll
                for (int i = 0; i < 2; ++i)
                    y[i] = dpp_move<ROW_SHL4, BANK_H0>(x[LOC[2 + i]], x[LOC[i]]) + dpp_move<ROW_SHR4, BANK_H1>(x[LOC[i]], x[LOC[2 + i]]);
                return dpp_move<ROW_ROR8, BANK_M0>(y[1], y[0]) + dpp_move<ROW_ROR8, BANK_M1>(y[0], y[1]);
            };
            const double cur1 = scatter_sum(fa1);
            const double cur0 = NEED_F0 ? scatter_sum(fa0) : 0.0;
            if (f > f0 && face_ok) {
                const double ihc = 0.25 * (STR ? a.ihc[f - 1] : a.inv_hn);  // 1/4: weight of a Gauss point
                const double d1 = (prev1 - cur1) * ihc, d0 = (prev0 - cur0) * ihc;
                if constexpr (MODE == 3) {
                    const long long xidx = 4 * rx_block_index(ce, je, ke, a.rx_nx, a.rx_nyb) + gvar;
                    a.rx1[xidx] = d1;
                    if (NEED_F0) a.rx0[xidx] = d0;
                } else if constexpr (MODE == 0) {
                    a.r1[ridx] = d1;
                    if (NEED_F0) a.r0[ridx] = d0;
                } else if constexpr (MODE == 5) {
                    out_a[pidx] = d1;
                    if (NEED_F0) out_b[pidx] = d0;
                } else {
                    const double L1 = r1v + (d1 + x1v), L0 = r0v + (d0 + x0v);
                    if (NEED_F0) {
                        out_a[pidx] = qe + 0.5 * dt * L0 + 0.125 * dt * dt * L1;
                        out_b[pidx] = qe + dt * L0 + (dt * dt * (1.0 / 6.0)) * L1;
                    } else {
                        out_a[pidx] = qe + ((dt * dt * (1.0 / 3.0)) * L1 + dt * gforce);
                    }
                }
            }
            prev1 = cur1;
            prev0 = cur0;
        }
        // the next march's column phase overwrites s_nrm, last read before the barrier above; s_t1 is
        // rewritten only after that phase's barrier
    }
}

// the launches: see the FP32 kernels of the same names
template <int T2, int STAGE, bool STR>
__global__ void __launch_bounds__(64 * T2) face64_xy_kernel(const FaceArgs<double> ax, const FaceArgs<double> ay) {
    __shared__ Face64Lds<T2 + 4> lds;
    const int nx = pad8(ax.n_wg), blk = blockIdx.x;
    if (blk < nx) face64_march<T2, STAGE, 3, STR>(ax, blk, nx, lds);
    else face64_march<T2, STAGE, 0, STR>(ay, blk - nx, pad8(ay.n_wg), lds);
}

template <int T2, int STAGE, bool STR>
__global__ void __launch_bounds__(64 * T2) face64_z_kernel(const FaceArgs<double> a) {
    __shared__ Face64Lds<T2 + 4> lds;
    if (STAGE == 2 && a.finish && blockIdx.x == 0 && threadIdx.x == 0) finish_step(a.finish);
    face64_march<T2, STAGE, 4, STR>(a, blockIdx.x, pad8(a.n_wg), lds);
}

template <int T2, int STAGE, bool STR>
__global__ void __launch_bounds__(64 * T2) face64_xyz_kernel(const FaceArgs<double> ax, const FaceArgs<double> ay,
                                                             const FaceArgs<double> az, const DtArgs dt) {
    __shared__ Face64Lds<T2 + 4> lds;
    const int nx = pad8(ax.n_wg), ny = pad8(ay.n_wg), blk = blockIdx.x;
    if (STAGE == 1 && blk == (int)gridDim.x - 1) {
        dt_update<64 * T2>(dt, reinterpret_cast<double*>(&lds.nrm));
        return;
    }
    if (blk < nx) face64_march<T2, STAGE, 3, STR>(ax, blk, nx, lds);
    else if (blk < nx + ny) face64_march<T2, STAGE, 0, STR>(ay, blk - nx, ny, lds);
    else face64_march<T2, STAGE, 5, STR>(az, blk - nx - ny, pad8(az.n_wg), lds);
}

template <int T2>
int slots64() {
    // workgroups of the face kernels that the device holds at once
    int dev = 0, cus = 0, per_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, face64_z_kernel<T2, 1, false>, 64 * T2, 0) != hipSuccess)
        return 0;
    return cus * per_cu;
}

template <>
int face_slots<double>(int t2) {
    return t2 == 12 ? slots64<12>() : slots64<8>();
}

#define GKS_LAUNCH_STR(KERNEL, T2, ST, BLOCKS, ...)                                                           \
    do {                                                                                                      \
        const dim3 grid((unsigned)(BLOCKS)), block(64 * T2);                                                  \
        if (str) hipLaunchKernelGGL((KERNEL<T2, ST, true>), grid, block, 0, s, __VA_ARGS__);                  \
        else hipLaunchKernelGGL((KERNEL<T2, ST, false>), grid, block, 0, s, __VA_ARGS__);                     \
        return hipGetLastError();                                                                             \
    } while (0)
#define GKS_LAUNCH64(KERNEL, ROWS, BLOCKS, ...)                                                               \
    do {                                                                                                      \
        if (ROWS == 12 && stage == 1) GKS_LAUNCH_STR(KERNEL, 12, 1, BLOCKS, __VA_ARGS__);                     \
        if (ROWS == 12) GKS_LAUNCH_STR(KERNEL, 12, 2, BLOCKS, __VA_ARGS__);                                   \
        if (ROWS == 8 && stage == 1) GKS_LAUNCH_STR(KERNEL, 8, 1, BLOCKS, __VA_ARGS__);                       \
        if (ROWS == 8) GKS_LAUNCH_STR(KERNEL, 8, 2, BLOCKS, __VA_ARGS__);                                     \
        return hipErrorInvalidValue;                                                                          \
    } while (0)

template <>
hipError_t launch_face_xy<double>(const FaceArgs<double>& ax, const FaceArgs<double>& ay, int stage, hipStream_t s) {
    const bool str = ax.stretched != 0;
    const long long blocks = (long long)pad8(ax.n_wg) + pad8(ay.n_wg);
    GKS_LAUNCH64(face64_xy_kernel, ax.t2, blocks, ax, ay);
}

template <>
hipError_t launch_face_z<double>(const FaceArgs<double>& a, int stage, hipStream_t s) {
    const bool str = a.stretched != 0;
    GKS_LAUNCH64(face64_z_kernel, a.t2, pad8(a.n_wg), a);
}

template <>
hipError_t launch_face_xyz<double>(const FaceArgs<double>& ax, const FaceArgs<double>& ay, const FaceArgs<double>& az,
                                   const DtArgs& dt, int stage, hipStream_t s) {
    const bool str = ax.stretched != 0;
    const long long blocks = (long long)pad8(ax.n_wg) + pad8(ay.n_wg) + pad8(az.n_wg) + (stage == 1 ? 1 : 0);
    GKS_LAUNCH64(face64_xyz_kernel, ax.t2, blocks, ax, ay, az, dt);
}

}  // namespace gks
