// gks_stage2.hip -- stages of the second-order GKS variant (the comparison scheme of the paper's accuracy
// study, Section 4.3.3; its construction is defined by reference only): the gas-kinetic flux and the S2O4
// stages of the high-order scheme, with van Leer-limited linear face states, central-difference gradients
// of the equilibrium state and one flux evaluation at the face centre.
//
// One launch does a whole stage: a workgroup of 512 threads owns 32 x 16 cells of the (x, y) plane (16 x 32 on
// grids of few cells in x) and marches along z; each thread evaluates the three lower (x, y) and upper (z) faces of
// its cell. The scheme reads 13 cells per face and does a few hundred operations on them, so it is bound by the passes
// over memory: one pass per direction (with residual arrays between them and a transposed copy of the field for the x
// pass) moved 590 MB per stage 1 of the 192 x 96 x 96 channel in FP32, this one 408 MB, where reading the state and
// writing the stage's results is 170 MB (the rest are halos and 10 to 27 spilled registers a lane). Four planes of the
// tile and its two-cell halo live in LDS (46 KB FP32, two workgroups per CU), the next plane is loaded a step ahead, the
// x and y fluxes of a plane are exchanged through LDS and the z flux is kept from one plane to the next. The faces at the
// tile's upper x and y ends are extra evaluations of two waves.
#include <type_traits>

#include "gks_internal.h"

namespace gks {

namespace {

constexpr int O2_THREADS = 512;

// Cells of a tile along x; along y it has O2_THREADS / this many. 16 on grids of up to 16 cells in x, which leave at
// least half of a 32-cell row idle (FP32, us a step with 32 / 16, and with a launch per direction on 16 x 16 tiles:
// 3 x 512 x 512 513 / 296, 424; 8 x 512 x 512 557 / 333, 571; 12 x 512 x 512 601 / 379, 676); 32 else, whose rows fill whole
// cache lines. The halo is as large either way (720 cells).
int stage2_tile_x(int nx) { return nx <= 16 ? 16 : 32; }

template <typename real>
__device__ __forceinline__ real van_leer(real dm, real dp) {
    const real prod = dm * dp;
    return prod > real(0) ? real(2) * prod * rcp<real>(dm + dp) : real(0);
}

template <typename real>
struct Vec4;
template <>
struct Vec4<float> {
    using type = float4;
};
template <>
struct Vec4<double> {
    using type = double4;
};

// global variable of each local one (density, normal, t1, t2 momenta) of the x, y, z faces
constexpr int kLocal[3][4] = {{0, 1, 2, 3}, {0, 2, 1, 3}, {0, 3, 1, 2}};

}  // namespace

template <typename real, int STAGE, bool STR, int O2X>
__global__ void __launch_bounds__(O2_THREADS, sizeof(real) == 4 ? 4 : 2) stage2_kernel(const Face2Args<real> a) {
    using V4 = typename Vec4<real>::type;
    constexpr int O2Y = O2_THREADS / O2X, O2H1 = O2X + 4, O2H2 = O2Y + 4;  // tile, and with two cells per side
    static_assert(O2X <= 64 && O2Y <= 64 && O2H1 * O2H2 <= 2 * O2_THREADS, "a wave per upper end, two cells a thread");
    constexpr bool NEED_F0 = (STAGE == 1);
    constexpr bool COMP = sizeof(real) == 4;   // FP32: compensated state in the stage update
    constexpr bool SHIFT = sizeof(real) == 4;  // FP32: normal momenta of a face as deviations from a workgroup constant
    constexpr int NF = NEED_F0 ? 2 : 1;
    __shared__ V4 s_q[4][O2H2][O2H1];       // planes, plane k in slot k mod 4
    __shared__ V4 s_fx[NF][O2Y][O2X + 1];   // fluxes of the lower x faces (F1, then F0)
    __shared__ V4 s_fy[NF][O2Y + 1][O2X];

    const int tid = threadIdx.x;
    if (STAGE == 2 && a.finish && blockIdx.x == 0 && tid == 0) finish_step(a.finish);
    // consecutive logical workgroups on the same XCD (grid padded to a multiple of 8)
    int b = (int)(blockIdx.x % 8) * (int)(gridDim.x / 8) + (int)(blockIdx.x / 8);
    const int nch = (a.n[2] + a.chunk - 1) / a.chunk;
    if (b >= a.tiles_x * a.tiles_y * nch) return;
    const int i0 = (b % a.tiles_x) * O2X;
    b /= a.tiles_x;
    const int j0 = (b % a.tiles_y) * O2Y;
    const int k0 = (b / a.tiles_y) * a.chunk;
    const int k1 = min(k0 + a.chunk, a.n[2]);

    const int ti = tid % O2X, tj = tid / O2X;
    const int i = i0 + ti, j = j0 + tj;
    const bool in = i < a.n[0] && j < a.n[1];
    // cells of a plane that this thread stages: positions tid and tid + 512 of the 720 ones, clamped to the
    // padded domain (what lies beyond reaches no cell of it)
    const int pos[2] = {tid, min(tid + O2_THREADS, O2H1 * O2H2 - 1)};
    long long src[2];
#pragma unroll
    for (int s = 0; s < 2; ++s)
        src[s] = a.pad0 + min(i0 - 2 + pos[s] % O2H1, a.n[0] + 2) +
                 (long long)min(j0 - 2 + pos[s] / O2H1, a.n[1] + 2) * a.st[1];
    auto load_plane = [&](int k, real (&x)[2][4]) {
        const long long off = (long long)min(k, a.n[2] + 2) * a.st[2];
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int v = 0; v < 4; ++v) x[s][v] = a.q[v][src[s] + off];
    };
    auto store_plane = [&](int k, const real (&x)[2][4]) {
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            V4 y;
            y.x = x[s][0];
            y.y = x[s][1];
            y.z = x[s][2];
            y.w = x[s][3];
            (&s_q[k & 3][0][0])[pos[s]] = y;
        }
    };
    // planes k0 - 2 .. k0 + 1 to LDS and k0 + 2 in registers, all loads issued together
    real nxt[2][4], pre[4][2][4];
#pragma unroll
    for (int r = 0; r < 4; ++r) load_plane(k0 - 2 + r, pre[r]);
    load_plane(k0 + 2, nxt);
    real cm[3] = {0, 0, 0};
    if constexpr (SHIFT) {
        // the midrange of each momentum over the domain's cells in the chunk's first plane of the tile (ghost cells
        // mirror a momentum at a wall, and the midrange would be zero in a stream towards it): the constant part of a mass
        // flux then cancels exactly between the two faces of a cell and FP32 rounding acts on the deviation only. The
        // planes in LDS keep the momenta whole: a tangential momentum much smaller than the midrange (at a no-slip
        // wall) would lose its low bits to the shift, and with them its derivatives
        __shared__ float s_range[6][O2_THREADS / 64];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            float lo = 3.0e38f, up = -3.0e38f;
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const int ci = i0 - 2 + pos[s] % O2H1, cj = j0 - 2 + pos[s] / O2H1;
                if (ci < 0 || ci >= a.n[0] || cj < 0 || cj >= a.n[1]) continue;
                lo = fminf(lo, pre[2][s][1 + d]);
                up = fmaxf(up, pre[2][s][1 + d]);
            }
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) {
                lo = fminf(lo, __shfl_xor(lo, o));
                up = fmaxf(up, __shfl_xor(up, o));
            }
            if ((tid & 63) == 0) {
                s_range[2 * d][tid >> 6] = lo;
                s_range[2 * d + 1][tid >> 6] = up;
            }
        }
        __syncthreads();
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            float lo = s_range[2 * d][0], up = s_range[2 * d + 1][0];
            for (int w = 1; w < O2_THREADS / 64; ++w) {
                lo = fminf(lo, s_range[2 * d][w]);
                up = fmaxf(up, s_range[2 * d + 1][w]);
            }
            cm[d] = 0.5f * (lo + up);
        }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) store_plane(k0 - 2 + r, pre[r]);

    // Flux of the face between cells -1 and 0 along axis D: at(n, t1, t2) is the cell at these offsets.
    auto face_flux = [&](auto dir, auto at, real ihf, real ih1, real ih2, V4& F1, V4& F0) {
        constexpr int D = decltype(dir)::value;
        const V4 cm2 = at(-2, 0, 0), cm1 = at(-1, 0, 0), c0 = at(0, 0, 0), cp1 = at(1, 0, 0);
        const V4 p1a = at(-1, 1, 0), p1b = at(0, 1, 0), m1a = at(-1, -1, 0), m1b = at(0, -1, 0);
        const V4 p2a = at(-1, 0, 1), p2b = at(0, 0, 1), m2a = at(-1, 0, -1), m2b = at(0, 0, -1);
        auto get = [](const V4& x, int v) { return v == 0 ? x.x : v == 1 ? x.y : v == 2 ? x.z : x.w; };
        real qL[4], qR[4], g[3][4], f0[4], f1[4];
#pragma unroll
        for (int l = 0; l < 4; ++l) {
            const int v = kLocal[D][l];
            const real qm2 = get(cm2, v), qm1 = get(cm1, v), q0 = get(c0, v), qp1 = get(cp1, v);
            const real dm = q0 - qm1;
            const real sh = SHIFT && l == 1 ? cm[D] : real(0);  // the normal momentum's deviation enters the flux
            qL[l] = (SHIFT && l == 1 ? qm1 - sh : qm1) + real(0.5) * van_leer(qm1 - qm2, dm);
            qR[l] = (SHIFT && l == 1 ? q0 - sh : q0) - real(0.5) * van_leer(dm, qp1 - q0);
            g[0][l] = dm * ihf;
            g[1][l] = ((get(p1a, v) + get(p1b, v)) - (get(m1a, v) + get(m1b, v))) * (real(0.25) * ih1);
            g[2][l] = ((get(p2a, v) + get(p2b, v)) - (get(m2a, v) + get(m2b, v))) * (real(0.25) * ih2);
        }
        gp_flux<real, NEED_F0, SHIFT>(qL, qR, g, a.fc, f0, f1, SHIFT ? cm[D] : real(0));
        auto put = [](V4& x, int v, real y) {
            if (v == 0) x.x = y;
            else if (v == 1) x.y = y;
            else if (v == 2) x.z = y;
            else x.w = y;
        };
#pragma unroll
        for (int l = 0; l < 4; ++l) {
            put(F1, kLocal[D][l], f1[l]);
            if (NEED_F0) put(F0, kLocal[D][l], f0[l]);
        }
    };

    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ic = min(i, a.n[0] - 1), jc = min(j, a.n[1] - 1);
    // inverse widths of this thread's cell and face spacings of its lower faces
    const real ihcx = STR ? a.ihc[0][ic] : a.inv_h[0], ihcy = STR ? a.ihc[1][jc] : a.inv_h[1];
    const real ihfx = STR ? a.ihf[0][min(i, a.n[0])] : a.inv_h[0], ihfy = STR ? a.ihf[1][min(j, a.n[1])] : a.inv_h[1];
    // the same at the tile's upper faces: x of row tid (wave 1), y of column tid (wave 0)
    const real ihfx_e = STR ? a.ihf[0][min(i0 + O2X, a.n[0])] : a.inv_h[0];
    const real ihfy_e = STR ? a.ihf[1][min(j0 + O2Y, a.n[1])] : a.inv_h[1];
    const int re = tid & 63;
    const real ihcy_e = STR ? a.ihc[1][min(j0 + min(re, O2Y - 1), a.n[1] - 1)] : a.inv_h[1];
    const real ihcx_e = STR ? a.ihc[0][min(i0 + min(re, O2X - 1), a.n[0] - 1)] : a.inv_h[0];
    const real dt = real(*a.dt_ptr);
    const long long pbase = a.pad0 + ic + (long long)jc * a.st[1];
    const long long cbase = ic + (long long)a.n[0] * jc;
    V4 zp1, zp0 = {};  // z fluxes of the face below
    __syncthreads();
    // step k evaluates the x and y faces of plane k and the z face above it; the step before the chunk only
    // the z face below its first plane
#pragma unroll 1
    for (int k = k0 - 1; k < k1; ++k) {
        const bool first = k < k0;
        const int sl[4] = {(k - 1) & 3, k & 3, (k + 1) & 3, (k + 2) & 3};
        const real ihcz = STR ? a.ihc[2][max(k, 0)] : a.inv_h[2];
        V4 X1, X0 = {}, Y1, Y0 = {};
        // epilogue operands of cell (i, j, k), loaded ahead of the plane's arithmetic
        const long long p = pbase + (long long)max(k, 0) * a.st[2];
        const long long c = cbase + (long long)a.n[0] * a.n[1] * max(k, 0);
        real qe[4];
        V4 lo = {};
#pragma unroll
        for (int v = 0; v < 4; ++v) qe[v] = NEED_F0 ? a.q_c[v][p] : a.s_in[v][p];
        if (COMP) lo = *reinterpret_cast<const V4*>(a.lo_in + 4 * c);
        if (!first) {
            // x faces: every thread's lower one; wave 1 then the 16 faces at the tile's upper end
#pragma unroll 1
            for (int rep = 0; rep < (wave == 1 ? 2 : 1); ++rep) {
                const int fi = rep ? O2X : ti, fj = rep ? min(re, O2Y - 1) : tj;
                V4 F1, F0 = {};
                face_flux(std::integral_constant<int, 0>{},
                          [&](int n, int y, int z) { return s_q[sl[1 + z]][fj + 2 + y][fi + 2 + n]; },
                          rep ? ihfx_e : ihfx, rep ? ihcy_e : ihcy, ihcz, F1, F0);
                if (rep == 0) {
                    X1 = F1;
                    X0 = F0;
                }
                if (rep == 0 || re < O2Y) {
                    s_fx[0][fj][fi] = F1;
                    if (NEED_F0) s_fx[NF - 1][fj][fi] = F0;
                }
            }
            // y faces: wave 0 then the 32 faces at the tile's upper end
#pragma unroll 1
            for (int rep = 0; rep < (wave == 0 ? 2 : 1); ++rep) {
                const int fi = rep ? min(re, O2X - 1) : ti, fj = rep ? O2Y : tj;
                V4 F1, F0 = {};
                face_flux(std::integral_constant<int, 1>{},
                          [&](int n, int x, int z) { return s_q[sl[1 + z]][fj + 2 + n][fi + 2 + x]; },
                          rep ? ihfy_e : ihfy, rep ? ihcx_e : ihcx, ihcz, F1, F0);
                if (rep == 0) {
                    Y1 = F1;
                    Y0 = F0;
                }
                if (rep == 0 || re < O2X) {
                    s_fy[0][fj][fi] = F1;
                    if (NEED_F0) s_fy[NF - 1][fj][fi] = F0;
                }
            }
        }
        V4 Z1, Z0 = {};
        face_flux(std::integral_constant<int, 2>{},
                  [&](int n, int x, int y) { return s_q[sl[2 + n]][tj + 2 + y][ti + 2 + x]; },
                  STR ? a.ihf[2][k + 1] : a.inv_h[2], ihcx, ihcy, Z1, Z0);
        __syncthreads();
        // plane k - 1 was last read before the barrier: plane k + 3 takes its slot
        store_plane(k + 3, nxt);
        load_plane(k + 4, nxt);
        if (!first && in) {
            const V4 xr1 = s_fx[0][tj][ti + 1], yr1 = s_fy[0][tj + 1][ti];
            V4 xr0 = {}, yr0 = {};
            if (NEED_F0) {
                xr0 = s_fx[NF - 1][tj][ti + 1];
                yr0 = s_fy[NF - 1][tj + 1][ti];
            }
            auto res = [&](real xl, real xr, real yl, real yr, real zl, real zr) {
                return (yl - yr) * ihcy + ((zl - zr) * ihcz + (xl - xr) * ihcx);
            };
            const real L1[4] = {res(X1.x, xr1.x, Y1.x, yr1.x, zp1.x, Z1.x), res(X1.y, xr1.y, Y1.y, yr1.y, zp1.y, Z1.y),
                                res(X1.z, xr1.z, Y1.z, yr1.z, zp1.z, Z1.z), res(X1.w, xr1.w, Y1.w, yr1.w, zp1.w, Z1.w)};
            const real L0[4] = {res(X0.x, xr0.x, Y0.x, yr0.x, zp0.x, Z0.x), res(X0.y, xr0.y, Y0.y, yr0.y, zp0.y, Z0.y),
                                res(X0.z, xr0.z, Y0.z, yr0.z, zp0.z, Z0.z), res(X0.w, xr0.w, Y0.w, yr0.w, zp0.w, Z0.w)};
            const real lov[4] = {lo.x, lo.y, lo.z, lo.w};
            real la[4], lb[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const real add = NEED_F0 ? real(0.5) * dt * L0[v] + real(0.125) * dt * dt * L1[v]
                                         : (dt * dt * real(1.0 / 3.0)) * L1[v] + (v > 0 ? dt * a.g_global[v > 0 ? v - 1 : 0] : real(0));
                const real add2 = NEED_F0 ? dt * L0[v] + (dt * dt * real(1.0 / 6.0)) * L1[v] : real(0);
                if constexpr (COMP) {
                    float sh, sl_;
                    two_sum(qe[v], lov[v] + add, sh, sl_);
                    a.out_a[v][p] = sh;
                    la[v] = sl_;
                    if (NEED_F0) {
                        two_sum(qe[v], lov[v] + add2, sh, sl_);
                        a.out_b[v][p] = sh;
                        lb[v] = sl_;
                    }
                } else {
                    a.out_a[v][p] = qe[v] + add;
                    if (NEED_F0) a.out_b[v][p] = qe[v] + add2;
                }
            }
            if constexpr (COMP) {
                *reinterpret_cast<V4*>(a.lo_a + 4 * c) = V4{la[0], la[1], la[2], la[3]};
                if (NEED_F0) *reinterpret_cast<V4*>(a.lo_b + 4 * c) = V4{lb[0], lb[1], lb[2], lb[3]};
            }
        }
        zp1 = Z1;
        zp0 = Z0;
        __syncthreads();
    }
}

int stage2_chunk(const int n[3], int f64) {
    // planes per workgroup: rounds of the resident workgroups times (planes + the start of a march)
    int dev = 0, cus = 0, per_cu = 0;
    int slots = 0;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess) {
        const hipError_t e =
            f64 ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, stage2_kernel<double, 1, false, 32>, O2_THREADS, 0)
                : hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, stage2_kernel<float, 1, false, 32>, O2_THREADS, 0);
        if (e == hipSuccess) slots = cus * per_cu;
    }
    const int tx = stage2_tile_x(n[0]), ty = O2_THREADS / tx;
    return face_chunk(n[2], ((n[0] + tx - 1) / tx) * ((n[1] + ty - 1) / ty), slots);
}

template <typename real, int O2X>
hipError_t launch_stage2_tiles(Face2Args<real> a, int stage, hipStream_t s) {
    constexpr int O2Y = O2_THREADS / O2X;
    a.tiles_x = (a.n[0] + O2X - 1) / O2X;
    a.tiles_y = (a.n[1] + O2Y - 1) / O2Y;
    const long long blocks = ((long long)a.tiles_x * a.tiles_y * ((a.n[2] + a.chunk - 1) / a.chunk) + 7) / 8 * 8;
    if (blocks <= 0 || blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    const dim3 grid((unsigned)blocks), block(O2_THREADS);
    if (stage == 1) {
        if (a.stretched) hipLaunchKernelGGL((stage2_kernel<real, 1, true, O2X>), grid, block, 0, s, a);
        else hipLaunchKernelGGL((stage2_kernel<real, 1, false, O2X>), grid, block, 0, s, a);
    } else {
        if (a.stretched) hipLaunchKernelGGL((stage2_kernel<real, 2, true, O2X>), grid, block, 0, s, a);
        else hipLaunchKernelGGL((stage2_kernel<real, 2, false, O2X>), grid, block, 0, s, a);
    }
    return hipGetLastError();
}

template <typename real>
hipError_t launch_stage2(const Face2Args<real>& a, int stage, hipStream_t s) {
    return stage2_tile_x(a.n[0]) == 16 ? launch_stage2_tiles<real, 16>(a, stage, s) : launch_stage2_tiles<real, 32>(a, stage, s);
}

template hipError_t launch_stage2<float>(const Face2Args<float>&, int, hipStream_t);
template hipError_t launch_stage2<double>(const Face2Args<double>&, int, hipStream_t);

}  // namespace gks
