// gks_adjoint.hip -- discrete adjoint of the S2O4 step (FP64) with the actuator-line body force, for
// the gradient of a rotor objective with respect to per-point force scalings.
//
// Forward operator per face direction (Section 2): normal WENO/derivative reconstruction ->
// t1 Gauss-point sweep -> t2 Gauss-point sweep -> gas-kinetic flux at the 2x2 Gauss points ->
// face quadrature and divergence. Its transpose is applied tile by tile in gather form (each output
// is one thread summing a fixed list of terms), with the WENO nonlinear weights frozen at their
// forward values or differentiated too; every other operator is linearised exactly. No atomics are
// used, so gradients are bitwise reproducible.
#include <algorithm>
#include <type_traits>

#include "gks.h"
#include "gks_adjoint.h"

namespace gks {

namespace {

// Coefficients of one WENO evaluation on `side` (stencil q, nonlinear weights w, value v): the frozen
// weights w0 and w2 (w1 = 1 - w0 - w2 is rebuilt where they are used) or (EXACT) the Jacobian row.
template <bool EXACT>
__device__ __forceinline__ void weno_coefs(int side, const double q[5], double eps, const double w[3], double v,
                                           double* out) {
    if constexpr (EXACT) {
        weno_jacobian(side, q, eps, w, v, out);
    } else {
        out[0] = w[0];
        out[1] = w[2];
    }
}

// Coefficient of stencil cell r in a WENO evaluation on `side` from its coefficients: the frozen weights
// expanded over the sub-stencils, or (EXACT) the Jacobian entry.
template <bool EXACT>
__device__ __forceinline__ double wcoef(int side, const double* c, int r) {
    if constexpr (EXACT) {
        return c[r];
    } else {
        const double w[3] = {c[0], 1.0 - c[0] - c[1], c[1]};
        return weno_eff(side, w, r);
    }
}

// The value of lane + K (shl) or lane - K (shr) of a row, zero where that lies outside it.
template <int K>
__device__ __forceinline__ double dpp_shl(double x) {
    return dpp_move<0x100 + K, 0xF, true>(0.0, x);
}
template <int K>
__device__ __forceinline__ double dpp_shr(double x) {
    return dpp_move<0x110 + K, 0xF, true>(0.0, x);
}

// Kernel arguments as they stand in the argument block, by a reference the compiler cannot see through: it then
// loads a field with a scalar load where it is used. With copies of them all, which spill into vector registers,
// adj_face_kernel keeps 7 dwords more in scratch: the 128^3 window of 20 steps took 174 ms, now 167. (The
// forward's FP64 kernels lose their 99 spilled scalars too, but wait for the loads: 32^3 2 % slower.)
template <typename T>
__device__ __forceinline__ const T& args_in_place(const T& a) {
    int zero = 0;
    asm("" : "+s"(zero));
    return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(&a) + zero);
}

}  // namespace

// ------------------------------------------------------------------------------------------------
// The tile's forward face pipeline and its transpose, down to the cells of the tile's columns.
//
// The kernel marches 16 x 8 face tiles with the lane layout of the forward FP64 kernel (four lanes per face:
// lane bit 2 is h, bit 3 m; a wave per t2 row) and, per face, runs the reverse of the flux at each Gauss point,
// undoes the exchange of the lane pair, and transposes the t2 sweep, the t1 sweep, C = (q^L + q^R)/2 and the
// normal reconstruction inside the tile. Only the adjoints of the cells of the tile's 20 x 12 columns leave it,
// partial sums in the two-cell halo and at the ends of a march, which adj_sum_kernel adds in a fixed order.
// With separate kernels the Gauss-point adjoints (640 B a face) and the inputs of the tangential WENO evaluations
// (192 B) went through memory, at 2.6 to 3.7 TB/s and one wave per SIMD: 1.95 ms per direction and stage of the
// 128^3 rotor box, against 0.79 ms and 0.07 ms of adj_sum_kernel. This one writes 60 B a face and is bound by FP64
// issue and its barriers.
//
// t2 transpose: each lane forms, for its two variables, the WENO terms of its face for the five rows it reaches
// (10 values) and keeps the linear terms' six inputs; these 16 values go to LDS (over the t1 results, then dead), and
// a thread per (variable, position, line) and run of three rows gathers the seven faces that reach them.
// t1 transpose: a lane per (variable, row, position) forms its terms for five columns; neighbouring positions are
// neighbouring lanes, so the sums over positions are DPP shifts inside the row of 16, the four columns beyond its ends
// landing in lanes 14, 15, 0 and 1.
// ------------------------------------------------------------------------------------------------
template <int STAGE, bool EXACT>
__global__ void __launch_bounds__(AdjTile::THREADS) adj_face_kernel(const AdjFaceArgs args) {
    const AdjFaceArgs& a = args_in_place(args);
    constexpr bool NEED_F0 = (STAGE == 1);
    constexpr int T2 = AdjTile::T2, X2 = T2 + 4, NTH = AdjTile::THREADS, NW = EXACT ? 5 : 2;
    static_assert(T2 == 8 && NTH == 64 * T2 && 2 * EXT1 * X2 <= NTH, "thread roles");
    // padded as in the forward kernel
    __shared__ struct {
        double a[4][X2][EXT1];
        double pad[16];
    } s_nrm[4];
    // t1 results, then the faces' terms of the t2 transpose, then the t1-line adjoints
    __shared__ double s_w[32 * NTH];
    // doubles per variable: variables v and v + 2 start 16 words apart modulo 32, so the 16 lanes of a t2-phase read
    // meet no bank twice (32 words apart: 128^3 window 167 ms, now 163; 48^3 field 2.73 ms, now 2.65)
    constexpr int T1S = 5 * X2 * 32 + 4;
    // adjoints of the normal face values [variable][q^L, q^R, D][t2 row][t1 column], beside the t1-line adjoints
    double* const s_fb = s_w + 4 * T1S;
    static_assert(4 * T1S + 12 * X2 * EXT1 <= 32 * NTH, "LDS regions");
    auto t1_at = [&](int v, int q, int row, int c) -> double& { return s_w[v * T1S + (q * X2 + row) * 32 + c]; };

    const int tid = threadIdx.x;
    const int b = (int)(blockIdx.x % 8) * (int)(gridDim.x / 8) + (int)(blockIdx.x / 8);
    if (b >= a.n_wg) return;
    // faces [f0, f1) of one tile
    const int nf = a.n_n + 1;
    const int tiles = a.tiles_t1 * a.tiles_t2;
    const double eps = a.eps;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    // column role: variables cv, cv + 1 of column (c1, c2)
    const int half = __builtin_amdgcn_readfirstlane(tid / (NTH / 2));
    const int cv = 2 * half, ct = tid % (NTH / 2);
    const bool col = ct < EXT1 * X2;
    const int c1 = ct % EXT1, c2 = ct / EXT1;
    const double* const qcol[2] = {half ? a.q[2] : a.q[0], half ? a.q[3] : a.q[1]};
    // face role
    const int hi = (tid >> 2) & 1, m = (tid >> 3) & 1;
    const int fj = (tid & 3) + 4 * ((tid >> 4) & 3), fk = wv;
    const int own = 2 * hi + m;  // the variable whose seeds this lane loads
    auto lane_field = [&](const double* const(&p)[4]) {
        return hi ? (m ? p[3] : p[2]) : (m ? p[1] : p[0]);
    };
    const double* const lam = lane_field(a.seed_lam);
    const double* const star = lane_field(a.seed_star);
    // the two seeds of a cell over its width
    auto seed = [&](long long idx, double w, double& m0, double& m1) {
        const double x = lam[idx] * w;
        m1 = a.lt[0] * x;
        if (NEED_F0) {
            const double y = star[idx] * w;
            m0 = a.l[0] * x + a.l[1] * y;
            m1 += a.lt[1] * y;
        }
    };
    // t1 role: position tj of variable tv
    const int tj = tid & 15, tv = (tid >> 4) & 3;

    {
        const int tile = b % tiles, f0 = (b / tiles) * a.chunk, f1 = min(f0 + a.chunk, nf);
        const int j0 = (tile % a.tiles_t1) * TILE1, k0 = (tile / a.tiles_t1) * T2;
        // columns outside the padded domain read a clamped column; their faces have zero seeds
        const int jc = min(j0 - 2 + c1, a.n_t1 + NG - 1), kc = min(k0 - 2 + min(c2, X2 - 1), a.n_t2 + NG - 1);
        const long long cbase = a.qpad0 + (long long)jc * a.qst_t1 + (long long)kc * a.qst_t2;
        const bool face_ok = (j0 + fj < a.n_t1) && (k0 + fk < a.n_t2);
        const int je = min(j0 + fj, a.n_t1 - 1), ke = min(k0 + fk, a.n_t2 - 1);
        const long long mbase = a.qpad0 + (long long)je * a.qst_t1 + (long long)ke * a.qst_t2;
        const double ih2 = a.ih2[ke], ih1 = a.ih1[min(j0 + tj, a.n_t1 - 1)];
        // cells f0-3 .. f0+1 and the next; of the evaluation on cell f0-1 its right value (q^L of face f0) and
        // that value's coefficients; the adjoints of cells f-3 .. f+2 that the faces so far reach
        double ring[2][5], carry[2], nxt[2], coefL[2][NW], cell[2][6];
#pragma unroll
        for (int v = 0; v < 2; ++v) {
#pragma unroll
            for (int r = 0; r < 5; ++r) ring[v][r] = qcol[v][cbase + (long long)(f0 - 3 + r) * a.qst_n];
            nxt[v] = qcol[v][cbase + (long long)min(f0 + 2, a.n_n + 2) * a.qst_n];
            double left, wr[3], wl[3];
            weno_faces_w<double>(ring[v][0], ring[v][1], ring[v][2], ring[v][3], ring[v][4], eps, carry[v], left, wr, wl);
            weno_coefs<EXACT>(0, ring[v], eps, wr, carry[v], coefL[v]);
#pragma unroll
            for (int r = 0; r < 6; ++r) cell[v][r] = 0.0;
        }
        // this march's cells f0-3 .. f1+1 of its columns, [cell][variable][column]
        const int var_len = a.x1 * a.x2;
        const bool keep = col && c1 < a.x1 && c2 < a.x2;
        double* slab = a.slab + ((long long)tile * a.nch + f0 / a.chunk) * (a.chunk + 5) * (4 * var_len) + cv * var_len +
                       c2 * a.x1 + c1;
        // seeds Fbar(f) = mu(f) / w_f - mu(f-1) / w_{f-1} (cell widths w; no cell beyond the ends) of this
        // lane's variable; the lower cell's term is kept from face to face
        double lo0 = 0.0, lo1 = 0.0;
        if (f0 >= 1) seed(mbase + (long long)(f0 - 1) * a.qst_n, a.ihc[f0 - 1], lo0, lo1);
        for (int f = f0; f < f1; ++f) {
            double up0 = 0.0, up1;
            {
                const int c = min(f, a.n_n - 1);
                seed(mbase + (long long)c * a.qst_n, f < a.n_n ? a.ihc[c] : 0.0, up0, up1);
            }
            // ---- column phase
            {
                const double ihf = a.ihf[f];
                const long long idx = cbase + (long long)min(f + 3, a.n_n + 2) * a.qst_n;
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
                                                     ((1.0 / 12.0) * ihf);
                        s_nrm[cv + v].a[3][c2][c1] = 0.5 * (qL + left);
                        carry[v] = right;
                    }
                }
            }
            __syncthreads();
            // ---- t1 phase
#pragma unroll
            for (int kk = 0; kk < (X2 + T2 - 1) / T2; ++kk) {
                const int tk = wv + kk * T2;
                if (tk < X2) {
                    double x[5], vm, vp;
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
#pragma unroll
                        for (int r = 0; r < 5; ++r) x[r] = s_nrm[tv].a[q][tk][tj + r];
                        if (q < 2) weno_gauss<double>(x[0], x[1], x[2], x[3], x[4], eps, vm, vp);
                        else quartic_gauss_value<double>(x[0], x[1], x[2], x[3], x[4], vm, vp);
                        t1_at(tv, q == 3 ? 4 : q, tk, 2 * tj) = vm;
                        t1_at(tv, q == 3 ? 4 : q, tk, 2 * tj + 1) = vp;
                        if (q == 3) {
                            quartic_gauss_deriv<double>(x[0], x[1], x[2], x[3], x[4], vm, vp);
                            t1_at(tv, 3, tk, 2 * tj) = vm * ih1;
                            t1_at(tv, 3, tk, 2 * tj + 1) = vp * ih1;
                        }
                    }
                }
            }
            __syncthreads();
            // ---- t2 phase: variables 2h, 2h + 1 of line m at both Gauss points, exchanged so that lane h holds
            // all four variables at point n = h
            double w[4][5];
            {
                double gp[2][2][5];
#pragma unroll
                for (int v = 0; v < 2; ++v)
#pragma unroll
                    for (int q = 0; q < 5; ++q) {
                        double y[5], vm, vp;
#pragma unroll
                        for (int r = 0; r < 5; ++r) y[r] = t1_at(2 * hi + v, q, fk + r, 2 * fj + m);
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
#pragma unroll
                for (int v = 0; v < 2; ++v)
#pragma unroll
                    for (int q = 0; q < 5; ++q) {
                        w[v][q] = dpp_move<ROW_SHR4, BANK_H1>(gp[v][0][q], gp[v][1][q]);
                        w[2 + v][q] = dpp_move<ROW_SHL4, BANK_H0>(gp[v][1][q], gp[v][0][q]);
                    }
            }
            // ---- reverse of the flux at this lane's Gauss point
            {
                // the four lanes of a face hold one seed each: all four to every lane
                auto all_lanes = [&](double x, double (&y)[4]) {
                    const double e = dpp_move<ROW_ROR8, BANK_M1>(x, x), o = dpp_move<ROW_ROR8, BANK_M0>(x, x);
                    y[0] = dpp_move<ROW_SHR4, BANK_H1>(e, e);
                    y[1] = dpp_move<ROW_SHR4, BANK_H1>(o, o);
                    y[2] = dpp_move<ROW_SHL4, BANK_H0>(e, e);
                    y[3] = dpp_move<ROW_SHL4, BANK_H0>(o, o);
                };
                double b0[4] = {0, 0, 0, 0}, b1[4];
                all_lanes(face_ok ? up1 - lo1 : 0.0, b1);
                if (NEED_F0) all_lanes(face_ok ? up0 - lo0 : 0.0, b0);
                lo1 = up1;
                lo0 = up0;
                double qL[4], qR[4], g[3][4], qLb[4] = {0, 0, 0, 0}, qRb[4] = {0, 0, 0, 0};
                double gb[3][4] = {{0, 0, 0, 0}, {0, 0, 0, 0}, {0, 0, 0, 0}};
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    qL[v] = w[v][0];
                    qR[v] = w[v][1];
                    g[0][v] = w[v][2];
                    g[1][v] = w[v][3];
                    g[2][v] = w[v][4];
                }
                gp_flux_adj<NEED_F0>(qL, qR, g, a.fc, 0.25, b0, b1, qLb, qRb, gb);
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    w[v][0] = qLb[v];
                    w[v][1] = qRb[v];
                    w[v][2] = gb[0][v];
                    w[v][3] = gb[1][v];
                    w[v][4] = gb[2][v];
                }
            }
            // ---- terms of the t2 transpose, variable by variable
            double term[2][16];
#pragma unroll
            for (int v = 0; v < 2; ++v) {
                double gn[2][5];  // the exchange undone: both Gauss points of variable 2h + v
#pragma unroll
                for (int q = 0; q < 5; ++q) {
                    gn[0][q] = dpp_move<ROW_SHR4, BANK_H1>(w[v][q], w[2 + v][q]);
                    gn[1][q] = dpp_move<ROW_SHL4, BANK_H0>(w[2 + v][q], w[v][q]);
                }
#pragma unroll
                for (int side = 0; side < 2; ++side) {
                    double y[5], vm, vp, wm[3], wp[3], cm[NW], cp[NW];
#pragma unroll
                    for (int r = 0; r < 5; ++r) y[r] = t1_at(2 * hi + v, side, fk + r, 2 * fj + m);
                    weno_gauss_w<double>(y[0], y[1], y[2], y[3], y[4], eps, vm, vp, wm, wp);
                    weno_coefs<EXACT>(2, y, eps, wm, vm, cm);
                    weno_coefs<EXACT>(3, y, eps, wp, vp, cp);
#pragma unroll
                    for (int r = 0; r < 5; ++r)
                        term[v][5 * side + r] = wcoef<EXACT>(2, cm, r) * gn[0][side] + wcoef<EXACT>(3, cp, r) * gn[1][side];
                }
#pragma unroll
                for (int q = 2; q < 5; ++q)
#pragma unroll
                    for (int n = 0; n < 2; ++n) term[v][10 + 2 * (q - 2) + n] = q == 4 ? gn[n][q] * ih2 : gn[n][q];
            }
            __syncthreads();
#pragma unroll
            for (int v = 0; v < 2; ++v)
#pragma unroll
                for (int k = 0; k < 16; ++k) s_w[(16 * v + k) * NTH + tid] = term[v][k];
            __syncthreads();
            // ---- t2 transpose: rows 3 run .. 3 run + 2 of variable 2h + (wave & 1), ascending faces
            double tb[3][5];
            {
                const int i = wv & 1, run = wv >> 1;
#pragma unroll
                for (int p = 0; p < 3; ++p)
#pragma unroll
                    for (int q = 0; q < 5; ++q) tb[p][q] = 0.0;
#pragma unroll
                for (int jf = 0; jf < 7; ++jf) {
                    const int k = 3 * run - 4 + jf;  // face row
                    if (k >= 0 && k < T2) {
                        const double* const t = s_w + (16 * i) * NTH + k * 64 + (tid & 63);
                        double g[6];
#pragma unroll
                        for (int n = 0; n < 6; ++n) g[n] = t[(10 + n) * NTH];
#pragma unroll
                        for (int p = 0; p < 3; ++p) {
                            const int r = p + 4 - jf;
                            if (r < 0 || r > 4) continue;
                            tb[p][0] += t[r * NTH];
                            tb[p][1] += t[(5 + r) * NTH];
                            tb[p][2] += quartic_coef(0, -1, r) * g[0] + quartic_coef(0, 1, r) * g[1];
                            tb[p][3] += quartic_coef(0, -1, r) * g[2] + quartic_coef(0, 1, r) * g[3];
                            tb[p][4] += quartic_coef(1, -1, r) * g[4] + quartic_coef(1, 1, r) * g[5];
                        }
                    }
                }
            }
            __syncthreads();
#pragma unroll
            for (int p = 0; p < 3; ++p)
#pragma unroll
                for (int q = 0; q < 5; ++q) t1_at(2 * hi + (wv & 1), q, 3 * (wv >> 1) + p, 2 * fj + m) = tb[p][q];
            __syncthreads();
            // ---- t1 transpose and C = (q^L + q^R)/2
#pragma unroll
            for (int kk = 0; kk < (X2 + T2 - 1) / T2; ++kk) {
                const int tk = wv + kk * T2;
                if (tk < X2) {
                    double P[3][5];
                    {
                        const double d0 = t1_at(tv, 3, tk, 2 * tj) * ih1, d1 = t1_at(tv, 3, tk, 2 * tj + 1) * ih1;
                        const double c0 = t1_at(tv, 4, tk, 2 * tj), c1_ = t1_at(tv, 4, tk, 2 * tj + 1);
                        const double n0 = t1_at(tv, 2, tk, 2 * tj), n1 = t1_at(tv, 2, tk, 2 * tj + 1);
#pragma unroll
                        for (int r = 0; r < 5; ++r) {
                            const double cm = quartic_coef(0, -1, r), cp = quartic_coef(0, 1, r);
                            const double Cb = 0.5 * ((quartic_coef(1, -1, r) * d0 + quartic_coef(1, 1, r) * d1) + (cm * c0 + cp * c1_));
                            P[0][r] = Cb;
                            P[1][r] = Cb;
                            P[2][r] = cm * n0 + cp * n1;
                        }
                    }
#pragma unroll
                    for (int side = 0; side < 2; ++side) {
                        double x[5], vm, vp, wm[3], wp[3], cm[NW], cp[NW];
#pragma unroll
                        for (int r = 0; r < 5; ++r) x[r] = s_nrm[tv].a[side][tk][tj + r];
                        weno_gauss_w<double>(x[0], x[1], x[2], x[3], x[4], eps, vm, vp, wm, wp);
                        weno_coefs<EXACT>(2, x, eps, wm, vm, cm);
                        weno_coefs<EXACT>(3, x, eps, wp, vp, cp);
                        const double t0 = t1_at(tv, side, tk, 2 * tj), t1 = t1_at(tv, side, tk, 2 * tj + 1);
#pragma unroll
                        for (int r = 0; r < 5; ++r) P[side][r] += wcoef<EXACT>(2, cm, r) * t0 + wcoef<EXACT>(3, cp, r) * t1;
                    }
                    // column tj + r: stencil slot r of position tj. Lane l sums column l + 2; lanes 14, 15, 0, 1
                    // also hold columns 0, 1, 18, 19
                    const int edge = tj >= 14 ? tj - 14 : tj + 18;
#pragma unroll
                    for (int q = 0; q < 3; ++q) {
                        const double mid = ((dpp_shr<2>(P[q][4]) + dpp_shr<1>(P[q][3])) + P[q][2]) +
                                           (dpp_shl<1>(P[q][1]) + dpp_shl<2>(P[q][0]));
                        const double end = (dpp_shr<14>(P[q][0]) + dpp_shr<15>(P[q][1])) +
                                           (dpp_shl<15>(P[q][3]) + dpp_shl<14>(P[q][4]));
                        double* const o = s_fb + ((3 * tv + q) * X2 + tk) * EXT1;
                        o[tj + 2] = mid;
                        if (tj < 2 || tj >= 14) o[edge] = end;
                    }
                }
            }
            __syncthreads();
            // ---- transpose of the normal reconstruction: this thread's column and variables. Face f reaches cells
            // f-3 .. f+1 through q^L, f-2 .. f+2 through q^R and f-2 .. f+1 through D; cell f-3 is then complete
            if (col) {
                const double ihf = a.ihf[f] * (1.0 / 12.0);
#pragma unroll
                for (int v = 0; v < 2; ++v) {
                    const double* const fb = s_fb + ((3 * (cv + v)) * X2) * EXT1 + ct;
                    const double bL = fb[0], bR = fb[X2 * EXT1], bD = fb[2 * X2 * EXT1] * ihf;
                    double right, left, wr[3], wl[3], cR[NW];
                    weno_faces_w<double>(ring[v][0], ring[v][1], ring[v][2], ring[v][3], ring[v][4], eps, right, left, wr, wl);
                    weno_coefs<EXACT>(1, ring[v], eps, wl, left, cR);
#pragma unroll
                    for (int r = 0; r < 5; ++r) {
                        cell[v][r] += wcoef<EXACT>(0, coefL[v], r) * bL;
                        cell[v][1 + r] += wcoef<EXACT>(1, cR, r) * bR;
                    }
                    cell[v][1] += bD;
                    cell[v][2] -= 15.0 * bD;
                    cell[v][3] += 15.0 * bD;
                    cell[v][4] -= bD;
                    weno_coefs<EXACT>(0, ring[v], eps, wr, right, coefL[v]);
                    if (keep) slab[v * var_len] = cell[v][0];
#pragma unroll
                    for (int r = 0; r < 5; ++r) cell[v][r] = cell[v][r + 1];
                    cell[v][5] = 0.0;
                }
                slab += 4 * var_len;
            }
            // the next face rewrites s_nrm at once (last read before the barrier) and s_fb after two barriers
        }
        if (keep)
#pragma unroll
            for (int v = 0; v < 2; ++v)
#pragma unroll
                for (int r = 0; r < 5; ++r) slab[(4 * r + v) * var_len] = cell[v][r];
    }
}

// ------------------------------------------------------------------------------------------------
// Sum of the tiles' and marches' shares into the padded cell adjoint: added to it, or (the first direction) stored
// over it, in the interior on top of lam + star where the directions complete lam^n. A workgroup takes 32 t1
// positions x 16 cells of the normal for one t2 position and variable: read along t1 (the slabs' fastest index),
// written along the axis of unit stride (the normal in the x direction) through LDS. The up to four tiles' shares
// of a cell are in flight together and the marches that reach a cell are found once per workgroup: with a loop over
// tiles and marches that divided for each cell, four cells a thread, it took 24 us a direction on 48^3 and 99 us on
// 128^3, now 9.5 and 69 us (128^3: 270 MB, 3.9 TB/s). 32 cells: 11.4 and 66 us; one cell a thread: 10.6 and 87 us.
// ------------------------------------------------------------------------------------------------
constexpr int ADJ_SUM_THREADS = 256, ADJ_SUM_CELLS = 16;

__global__ void __launch_bounds__(ADJ_SUM_THREADS) adj_sum_kernel(const AdjFaceArgs a, int n_wg) {
    constexpr int X2 = AdjTile::T2 + 4, NI = ADJ_SUM_CELLS, RS = ADJ_SUM_THREADS / 32, NR = NI / RS;
    __shared__ double s_t[NI][33];
    const int nt1 = (a.n_t1 + 4 + 31) / 32, nn = (a.n_n + 6 + NI - 1) / NI;
    int b = (int)(blockIdx.x % 8) * (int)(gridDim.x / 8) + (int)(blockIdx.x / 8);
    if (b >= n_wg) return;
    const int jx0 = (b % nt1) * 32 - 2;
    b /= nt1;
    const int i0 = (b % nn) * NI - 3;
    b /= nn;
    const int v = b % 4, kx = b / 4 - 2;
    const int lane = threadIdx.x & 31, row = threadIdx.x >> 5;
    const int nf = a.n_n + 1;
    // marches whose faces reach cell i: faces i - 2 .. i + 3
    __shared__ int s_m[NI][2];
    if (threadIdx.x < NI) {
        const int i = i0 + (int)threadIdx.x;
        s_m[threadIdx.x][0] = max(i - 2, 0) / a.chunk;
        s_m[threadIdx.x][1] = min(i + 3, a.n_n) / a.chunk;
    }
    __syncthreads();
    {
        const int jx = jx0 + lane;
        // the tiles whose columns hold (jx, kx): in t1 and t2 the one before (its last four columns), then the own
        const int T1 = (jx + 2) / TILE1, c1 = (jx + 2) % TILE1, T2 = (kx + 2) / AdjTile::T2, c2 = (kx + 2) % AdjTile::T2;
        const int var_len = a.x1 * a.x2;
        const long long tile_len = (long long)a.nch * (a.chunk + 5) * (4 * var_len);
        const double* p[4];
        bool ok[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int d1 = 1 - (e & 1), d2 = 1 - (e >> 1);
            const int t1 = T1 - d1, t2 = T2 - d2;
            ok[e] = jx < a.n_t1 + 2 && t1 >= 0 && t1 < a.tiles_t1 && (d1 == 0 || c1 < EXT1 - TILE1) && t2 >= 0 &&
                    t2 < a.tiles_t2 && (d2 == 0 || c2 < X2 - AdjTile::T2);
            p[e] = a.slab + ((long long)t2 * a.tiles_t1 + t1) * tile_len + v * var_len + (c2 + AdjTile::T2 * d2) * a.x1 + c1 +
                   TILE1 * d1;
        }
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            const int i = i0 + row + RS * r;
            double sum = 0.0;
            if (i < a.n_n + 3) {
                for (int m = s_m[row + RS * r][0]; m <= s_m[row + RS * r][1]; ++m) {
                    const int f0 = m * a.chunk, len = min(a.chunk, nf - f0), slot = i - (f0 - 3);
                    if (slot < 0 || slot >= len + 5) continue;
                    const long long o = ((long long)m * (a.chunk + 5) + slot) * (4 * var_len);
                    double x[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (ok[e]) x[e] = p[e][o];
                    sum += (x[0] + x[1]) + (x[2] + x[3]);
                }
            }
            s_t[row + RS * r][lane] = sum;
        }
    }
    __syncthreads();
    const bool along_n = a.st_n == 1;
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        const int t = threadIdx.x + ADJ_SUM_THREADS * r;
        const int i = i0 + (along_n ? t % NI : t / 32), jx = jx0 + (along_n ? t / NI : t % 32);
        if (jx < a.n_t1 + 2 && i < a.n_n + 3) {
            const long long p = a.pad0 + (long long)i * a.st_n + (long long)jx * a.st_t1 + (long long)kx * a.st_t2;
            double base = 0.0;
            if (a.sum == ADJ_SUM_ACC) base = a.acc[v][p];
            else if (a.sum == ADJ_SUM_LAM_STAR && i >= 0 && i < a.n_n && jx >= 0 && jx < a.n_t1 && kx >= 0 && kx < a.n_t2)
                base = a.lam[v][p] + a.star[v][p];
            a.acc[v][p] = base + s_t[i - i0][jx - jx0];
        }
    }
}

template <bool EXACT>
hipError_t launch_adj_passes(const AdjFaceArgs& a, int stage, hipStream_t s) {
    if (a.n_wg <= 0) return hipErrorInvalidValue;
    const dim3 fgrid((unsigned)pad8(a.n_wg)), fblock(AdjTile::THREADS);
    if (stage == 1) hipLaunchKernelGGL((adj_face_kernel<1, EXACT>), fgrid, fblock, 0, s, a);
    else hipLaunchKernelGGL((adj_face_kernel<2, EXACT>), fgrid, fblock, 0, s, a);
    const long long blocks = (long long)((a.n_t1 + 4 + 31) / 32) * ((a.n_n + 6 + ADJ_SUM_CELLS - 1) / ADJ_SUM_CELLS) * 4 * (a.n_t2 + 4);
    if (blocks > 0x7fffffffLL - 7) return hipErrorInvalidValue;
    hipLaunchKernelGGL(adj_sum_kernel, dim3(pad8((int)blocks)), dim3(ADJ_SUM_THREADS), 0, s, a, (int)blocks);
    return hipGetLastError();
}

hipError_t launch_adj_direction(const AdjFaceArgs& a, int stage, hipStream_t s) {
    return a.exact ? launch_adj_passes<true>(a, stage, s) : launch_adj_passes<false>(a, stage, s);
}

// ------------------------------------------------------------------------------------------------
// transpose of the ghost fill: axes in reverse order (z, y, x); each thread folds the six ghost cells
// of one line and variable in a fixed order (a wave per variable: the ghost values of a side are in flight
// together, and inflow sides read all four variables before any is cleared)
// ------------------------------------------------------------------------------------------------
struct FoldArgs {
    int axis, n, np1, np2;
    long long st_a, st_1, st_2;
    int bc_lo, bc_hi;
    // inflow sides: the prescribed velocity, the sound speed, rho_ref and the padded field the ghost fill
    // was applied to (global variable order), at which the fill is linearised
    double u_in[3], c, rho_ref;
    Field4<const double> q;
};

__global__ void __launch_bounds__(256) adj_fold_kernel(Field4<double> f, FoldArgs g) {
    const int v = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const long long t = (long long)blockIdx.x * 64 + (threadIdx.x & 63);
    const bool ok = t < (long long)g.np1 * g.np2;
    const long long base = (t % g.np1) * g.st_1 + (t / g.np1) * g.st_2;
    double* const fv = f.v[v];
    auto at = [&](int i) { return base + (long long)(i + 3) * g.st_a; };  // cell i, 0 .. n - 1 inside
    auto ghost = [&](int side, int layer) { return at(side == 0 ? -1 - layer : g.n + layer); };
    double d[2][3];
    if (ok)
#pragma unroll
        for (int side = 0; side < 2; ++side)
#pragma unroll
            for (int layer = 0; layer < 3; ++layer) {
                const long long p = ghost(side, layer);
                d[side][layer] = (side == 0 ? g.bc_lo : g.bc_hi) != GKS_BC_INFLOW
                                     ? fv[p]
                                     : f.v[0][p] + g.u_in[0] * f.v[1][p] + g.u_in[1] * f.v[2][p] + g.u_in[2] * f.v[3][p];
            }
    __syncthreads();
    if (!ok) return;
    for (int side = 0; side < 2; ++side) {
        const int kind = side == 0 ? g.bc_lo : g.bc_hi;
#pragma unroll
        for (int layer = 0; layer < 3; ++layer) fv[ghost(side, layer)] = 0.0;
        if (kind == GKS_BC_INFLOW || kind == GKS_BC_OUTFLOW) {
            const long long src = at(side == 0 ? 0 : g.n - 1);
            double w = 1.0;
            if (kind == GKS_BC_INFLOW) {
                // ghost = (rho_g - rho_ref, rho_g u_in) with rho_g = rho_i e^x, x = s (u_in,n - m_n / rho_i) / C
                // (s = +1 on the low side, -1 on the high side): only rho' and m_n of the source enter,
                // d rho_g / d rho' = e^x (1 + s u_n / C), d rho_g / d m_n = -s e^x / C
                if (v != 0 && v != 1 + g.axis) continue;
                const double sgn = side == 0 ? 1.0 : -1.0;
                const double un = g.q.v[1 + g.axis][src] / (g.rho_ref + g.q.v[0][src]);
                const double ex = exp(sgn * (g.u_in[g.axis] - un) / g.c);
                w = v == 0 ? ex * (1.0 + sgn * un / g.c) : -sgn * ex / g.c;
            }
            double x = fv[src];
#pragma unroll
            for (int layer = 0; layer < 3; ++layer) x += w * d[side][layer];
            fv[src] = x;
        } else {
            const bool odd = (kind == GKS_BC_NOSLIP_WALL && v > 0) || (kind == GKS_BC_SLIP_WALL && v == 1 + g.axis);
            const bool low = (side == 0) != (kind == GKS_BC_PERIODIC);  // periodic: from the other end
            double x[3];
#pragma unroll
            for (int layer = 0; layer < 3; ++layer) x[layer] = fv[at(low ? layer : g.n - 1 - layer)];
#pragma unroll
            for (int layer = 0; layer < 3; ++layer)
                fv[at(low ? layer : g.n - 1 - layer)] = x[layer] + (odd ? -d[side][layer] : d[side][layer]);
        }
    }
}

hipError_t launch_adj_fold(double* fp[4], const GridDesc& gd, const int bc[6], const double* const q[4],
                           const double u_in[3], double c, double rho_ref, hipStream_t s) {
    Field4<double> f;
    for (int v = 0; v < 4; ++v) f.v[v] = fp[v];
    for (int axis = 2; axis >= 0; --axis) {
        FoldArgs g;
        g.axis = axis;
        g.n = gd.n[axis];
        const int a1 = axis == 0 ? 1 : 0, a2 = axis == 2 ? 1 : 2;
        g.np1 = gd.n[a1] + 6;
        g.np2 = gd.n[a2] + 6;
        g.st_a = gd.st[axis];
        g.st_1 = gd.st[a1];
        g.st_2 = gd.st[a2];
        g.bc_lo = bc[2 * axis];
        g.bc_hi = bc[2 * axis + 1];
        for (int j = 0; j < 3; ++j) g.u_in[j] = u_in[j];
        g.c = c;
        g.rho_ref = rho_ref;
        for (int v = 0; v < 4; ++v) g.q.v[v] = q[v];
        const long long total = (long long)g.np1 * g.np2;
        hipLaunchKernelGGL(adj_fold_kernel, dim3((unsigned)((total + 63) / 64)), dim3(256), 0, s, f, g);
    }
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// elementwise helpers
// ------------------------------------------------------------------------------------------------
__global__ void __launch_bounds__(256) interior_kernel(double* dst, Field4<const double> src, GridDesc g) {
    const long long n = (long long)g.n[0] * g.n[1] * g.n[2];
    const long long c = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= n) return;
    const int i = (int)(c % g.n[0]);
    const long long r = c / g.n[0];
    const int j = (int)(r % g.n[1]);
    const int k = (int)(r / g.n[1]);
    const long long p = g.pad0 + i * g.st[0] + j * g.st[1] + (long long)k * g.st[2];
#pragma unroll
    for (int v = 0; v < 4; ++v) dst[v * n + c] = src.v[v][p];
}

hipError_t launch_interior(double* dst, const double* const src[4], const GridDesc& g, hipStream_t s) {
    const long long n = (long long)g.n[0] * g.n[1] * g.n[2];
    Field4<const double> f;
    for (int v = 0; v < 4; ++v) f.v[v] = src[v];
    hipLaunchKernelGGL(interior_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, dst, f, g);
    return hipGetLastError();
}

// The [x][z][y] copies that the tile kernel's x direction reads: along x in the fields themselves each column and
// face keeps a line of its own in use, more than the L2s hold (128^3, stage 1: 1135 us against 825 of the other
// directions, with the copies 830; 48^3 113 and 91). A copy is bound by memory: 30 to 52 us on 128^3,
// 5.8 us on 48^3.
__global__ void __launch_bounds__(512) adj_transpose_kernel(Field4<double> dst, Field4<const double> src, int X, int Y, int Z,
                                                            int n_wg) {
    __shared__ double t[4][32][33];
    const int blk = (int)(blockIdx.x % 8) * (int)(gridDim.x / 8) + (int)(blockIdx.x / 8);
    if (blk >= n_wg) return;
    const int nbx = (X + 31) / 32, x0 = blk % nbx * 32, z = blk / nbx % Z, y0 = blk / nbx / Z * 32;
    const int lane = threadIdx.x & 31, row = threadIdx.x >> 5;
    double v[4][2];
#pragma unroll
    for (int w = 0; w < 4; ++w)
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int x = min(x0 + lane, X - 1), y = min(y0 + row + 16 * i, Y - 1);
            v[w][i] = src.v[w][((long long)z * Y + y) * X + x];
        }
#pragma unroll
    for (int w = 0; w < 4; ++w)
#pragma unroll
        for (int i = 0; i < 2; ++i) t[w][row + 16 * i][lane] = v[w][i];
    __syncthreads();
#pragma unroll
    for (int w = 0; w < 4; ++w)
#pragma unroll
        for (int i = row; i < 32; i += 16)
            if (x0 + i < X && y0 + lane < Y) dst.v[w][((long long)(x0 + i) * Z + z) * Y + y0 + lane] = t[w][lane][i];
}

hipError_t launch_adj_transpose(double* const dst[4], const double* const src[4], const GridDesc& g, hipStream_t s) {
    Field4<double> d;
    Field4<const double> f;
    for (int v = 0; v < 4; ++v) d.v[v] = dst[v], f.v[v] = src[v];
    const int X = g.n[0] + 6, Y = g.n[1] + 6, Z = g.n[2] + 6;
    const long long blocks = (long long)((X + 31) / 32) * ((Y + 31) / 32) * Z;
    if (blocks > 0x7fffffffLL - 7) return hipErrorInvalidValue;
    hipLaunchKernelGGL(adj_transpose_kernel, dim3(pad8((int)blocks)), dim3(512), 0, s, d, f, X, Y, Z, (int)blocks);
    return hipGetLastError();
}

__global__ void zero_kernel(double* y, long long n) {
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) y[i] = 0.0;
}

hipError_t launch_zero(double* y, long long n, hipStream_t s) {
    hipLaunchKernelGGL(zero_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, y, n);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// immersed-body adjoint (body at rest). Per forced cell the S direct-forcing iterations are affine in
// (rho, m): m^{s+1} = m^s + r (rho v-bar - m^s), r = V-bar / |Omega|, with V-bar and v-bar fixed by the
// body. Their transpose, taken through the iterations in reverse order, scales the momentum adjoint by
// (1 - r) per iteration and adds r v-bar . lambda_m to the density adjoint (the density is not forced).
// Every forced cell appears once in the body's cell list, so the cells are independent.
// ------------------------------------------------------------------------------------------------
__global__ void __launch_bounds__(256) ibm_adj_kernel(Field4<double> lam, IbmArgs a) {
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= a.ncell) return;
    const long long q = a.g.pad0 + (long long)a.cell[3 * c] * a.g.st[0] + (long long)a.cell[3 * c + 1] * a.g.st[1] +
                        (long long)a.cell[3 * c + 2] * a.g.st[2];
    const double r = a.vbar[c] / (a.g.h[0] * a.g.h[1] * a.g.h[2]);
    const double vv[3] = {a.vbar_vel[3 * c], a.vbar_vel[3 * c + 1], a.vbar_vel[3 * c + 2]};
    double lm[3] = {lam.v[1][q], lam.v[2][q], lam.v[3][q]};
    double lr = lam.v[0][q];
    for (int s = 0; s < a.iters; ++s) {
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            lr += r * vv[d] * lm[d];
            lm[d] *= 1.0 - r;
        }
    }
    lam.v[0][q] = lr;
#pragma unroll
    for (int d = 0; d < 3; ++d) lam.v[1 + d][q] = lm[d];
}

hipError_t launch_ibm_adjoint(double* lam[4], const IbmArgs& a, hipStream_t s) {
    if (a.moving || a.ncell_dev) return hipErrorInvalidValue;
    if (a.ncell <= 0 || a.iters <= 0) return hipSuccess;
    Field4<double> f;
    for (int v = 0; v < 4; ++v) f.v[v] = lam[v];
    hipLaunchKernelGGL(ibm_adj_kernel, dim3((unsigned)((a.ncell + 255) / 256)), dim3(256), 0, s, f, a);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// actuator-line adjoint
// ------------------------------------------------------------------------------------------------
__device__ __forceinline__ long long pidx_g(const GridDesc& g, int i, int j, int k) {
    return g.pad0 + (long long)i * g.st[0] + (long long)j * g.st[1] + (long long)k * g.st[2];
}

// per point: fvbar = dt sum_cells G(x - X_p) lambda_m(x) over the projection sphere; one workgroup per
// point, its threads striding over the cells of the sphere's bounding box, then a fixed-order tree sum
__global__ void __launch_bounds__(256) alm_adj_gather_kernel(AlmAdjArgs A) {
    const AlmArgs& a = A.fwd;
    const int p = blockIdx.x;  // uniform over the workgroup
    if (p >= a.n_act) return;
    const double X[3] = {a.X[3 * p], a.X[3 * p + 1], a.X[3 * p + 2]};
    const double cut = 9.0 * a.eps * a.eps, ie2 = 1.0 / (a.eps * a.eps);
    const double norm = 1.0 / (a.eps * a.eps * a.eps * M_PI * sqrt(M_PI));
    int lo[3], hi[3];
    for (int d = 0; d < 3; ++d) {
        lo[d] = (int)ceil((X[d] - 3.0 * a.eps - a.g.x0[d]) / a.g.h[d] - 0.5);
        hi[d] = (int)floor((X[d] + 3.0 * a.eps - a.g.x0[d]) / a.g.h[d] - 0.5);
        lo[d] = max(lo[d], a.box_lo[d]);
        hi[d] = min(hi[d], a.box_lo[d] + a.box_n[d] - 1);
    }
    const int nx = hi[0] - lo[0] + 1, ny = hi[1] - lo[1] + 1, nz = hi[2] - lo[2] + 1;
    const int ncell = (nx > 0 && ny > 0 && nz > 0) ? nx * ny * nz : 0;
    double acc[3] = {0, 0, 0};
    for (int c = threadIdx.x; c < ncell; c += blockDim.x) {
        const int i = lo[0] + c % nx, r = c / nx;
        const int j = lo[1] + r % ny, k = lo[2] + r / ny;
        const double dx = a.g.x0[0] + (i + 0.5) * a.g.h[0] - X[0];
        const double dy = a.g.x0[1] + (j + 0.5) * a.g.h[1] - X[1];
        const double dz = a.g.x0[2] + (k + 0.5) * a.g.h[2] - X[2];
        const double r2 = dx * dx + dy * dy + dz * dz;
        if (r2 <= cut) {
            const double gw = norm * exp(-r2 * ie2);
            const long long q = pidx_g(a.g, i, j, k);
            for (int d = 0; d < 3; ++d) acc[d] += gw * A.lam[1 + d][q];
        }
    }
    __shared__ double red[3][256];
    for (int d = 0; d < 3; ++d) red[d][threadIdx.x] = acc[d];
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w)
            for (int d = 0; d < 3; ++d) red[d][threadIdx.x] += red[d][threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const double dt = a.st->dt;
        for (int d = 0; d < 3; ++d) A.pt[d * a.n_act + p] = dt * red[d][0];
    }
}

// per point: reverse of the blade-element forces; gradient in s and the adjoint of the sampled U
__global__ void alm_adj_points_kernel(AlmAdjArgs A) {
    const AlmArgs& a = A.fwd;
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= a.n_act) return;
    const int bl = p / a.npb, ip = p % a.npb;
    const double t = a.st->t_next;
    const double th = a.theta0 + a.omega * t + 2.0 * M_PI * (double)bl / (double)a.nb;
    const double et1 = -sin(th), et2 = cos(th);
    const double rr = a.r[ip], chord = a.chord[ip], twist = a.twist[ip], width = a.width[ip];
    const double om = a.omega;
    const double U0 = a.out_u[3 * p], U1 = a.out_u[3 * p + 1], U2 = a.out_u[3 * p + 2];
    const double ux0 = U0, ut0 = U1 * et1 + U2 * et2;
    // forward recompute
    double ux = ux0, ut = ut0, fac = 1.0, g = 1.0, al0 = 0.0, U2_0 = 0.0;
    const double kc = chord / (4.0 * sqrt(M_PI) * a.eps);
    if (a.corr) {
        const double x0 = om * rr - ut0;
        U2_0 = ux0 * ux0 + x0 * x0;
        al0 = atan2(ux0, x0) - twist;
        const double cd0 = a.cd0 + a.cd2 * al0 * al0;
        g = 1.0 - cd0 * kc;
        fac = 1.0 / g;
        ux = ux0 * fac;
        ut = ut0 * fac;
    }
    const double xx = om * rr - ut;
    const double phi = atan2(ux, xx);
    const double alpha = phi - twist;
    const double wr = ut - om * rr;
    const double U2r = ux * ux + wr * wr;
    const bool inside = (alpha > -a.alpha_clip) && (alpha < a.alpha_clip);
    const double alc = fmin(fmax(alpha, -a.alpha_clip), a.alpha_clip);
    const double cl = a.cl_slope * alc, cd = a.cd0 + a.cd2 * alpha * alpha;
    const double q = 0.5 * a.rho_ref * chord * width * U2r;
    const double L = q * cl, D = q * cd;
    const double cph = cos(phi), sph = sin(phi);
    const double X0 = L * cph + D * sph, Y0 = L * sph - D * cph;
    double fa = 1.0, ftn = 1.0, dfa = 0.0, dft = 0.0;
    if (a.tip) {
        fa = tip_factor(a.g1_axi, a.nb, a.radius, rr, phi, &dfa);
        ftn = tip_factor(a.g1_tan, a.nb, a.radius, rr, phi, &dft);
    }
    const double fx0 = fa * X0, ft0 = ftn * Y0;
    const double sp = a.scale ? a.scale[p] : 1.0;
    // reverse
    const double fv0 = A.pt[p], fv1 = A.pt[a.n_act + p], fv2 = A.pt[2 * a.n_act + p];
    const double fxb = -fv0 + A.w1 * A.inv_n;
    const double ftb = -(fv1 * et1 + fv2 * et2) + A.w0 * A.inv_n * om * rr;
    A.grad_s[p] += fxb * fx0 + ftb * ft0;
    const double fx0b = sp * fxb, ft0b = sp * ftb;
    const double X0b = fx0b * fa, Y0b = ft0b * ftn;
    const double Lb = X0b * cph + Y0b * sph;
    const double Db = X0b * sph - Y0b * cph;
    double phib = -X0b * Y0 + Y0b * X0 + fx0b * X0 * dfa + ft0b * Y0 * dft;
    const double qb = Lb * cl + Db * cd;
    const double clb = Lb * q, cdb = Db * q;
    const double alb = clb * a.cl_slope * (inside ? 1.0 : 0.0) + cdb * 2.0 * a.cd2 * alpha;
    phib += alb;
    const double U2b = qb * 0.5 * a.rho_ref * chord * width;
    double uxb = U2b * 2.0 * ux + phib * xx / U2r;
    double utb = U2b * 2.0 * wr + phib * ux / U2r;
    if (a.corr) {
        const double facb = uxb * ux0 + utb * ut0;
        uxb *= fac;
        utb *= fac;
        const double gb = -facb / (g * g);
        const double cd0b = -gb * kc;
        const double al0b = cd0b * 2.0 * a.cd2 * al0;
        const double x0 = om * rr - ut0;
        uxb += al0b * x0 / U2_0;
        utb += al0b * ux0 / U2_0;
    }
    A.pt[3 * a.n_act + p] = uxb;
    A.pt[4 * a.n_act + p] = utb * et1;
    A.pt[5 * a.n_act + p] = utb * et2;
}

// adjoint of the velocity sampling (trilinear, or the mean of trilinear samples along the direction of
// motion) in gather form: one thread per cell of the sampling box adds, for the points in ascending
// order and their samples in ascending order, the terms of every sample whose eight trilinear cells
// hold it (the order of a serial sweep over points, samples and corners). Bound by the test of every sample in
// every cell: the workgroup places 256 samples at a time in LDS (each thread placing all of them, with two
// trigonometric functions and three divisions a sample, took 39 us for 48 points on 48^3 cells and 78 us for 96 on 128^3,
// against 14 and 18 us)
__global__ void __launch_bounds__(256) alm_adj_scatter_kernel(AlmAdjArgs A) {
    const AlmArgs& a = A.fwd;
    __shared__ int s_i[3][256];
    __shared__ double s_w[3][256], s_u[3][256];
    const long long ncell = (long long)a.samp_n[0] * a.samp_n[1] * a.samp_n[2];
    const long long tcell = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const bool ok = tcell < ncell;
    const int ci = a.samp_lo[0] + (int)(tcell % a.samp_n[0]);
    const int cj = a.samp_lo[1] + (int)((tcell / a.samp_n[0]) % a.samp_n[1]);
    const int ck = a.samp_lo[2] + (int)(tcell / ((long long)a.samp_n[0] * a.samp_n[1]));
    const long long q = pidx_g(a.g, ci, cj, ck);
    double rho = 0.0, Uc[3] = {0.0, 0.0, 0.0}, lam[4] = {0.0, 0.0, 0.0, 0.0};
    if (ok) {
        rho = a.rho_ref + A.qpre[0][q];
        for (int c = 0; c < 3; ++c) Uc[c] = A.qpre[1 + c][q] / rho;
        for (int v = 0; v < 4; ++v) lam[v] = A.lam[v][q];
    }
    bool touched = false;
    const int ns = a.line_n > 1 ? a.line_n : 1;
    const long long nsamp = (long long)a.n_act * ns;
    for (long long s0 = 0; s0 < nsamp; s0 += 256) {
        const int cnt = (int)min(256LL, nsamp - s0);
        __syncthreads();
        if ((int)threadIdx.x < cnt) {
            const int p = (int)((s0 + threadIdx.x) / ns), k = (int)((s0 + threadIdx.x) % ns), bl = p / a.npb;
            const double th = a.theta0 + a.omega * a.st->t_next + 2.0 * M_PI * (double)bl / (double)a.nb;
            const double sk = ns > 1 ? line_offset(a, k) : 0.0;
            const double Xs[3] = {a.X[3 * p], a.X[3 * p + 1] + sk * -sin(th), a.X[3 * p + 2] + sk * cos(th)};
            for (int d = 0; d < 3; ++d) {
                const double fc = (Xs[d] - a.g.x0[d]) / a.g.h[d] - 0.5;
                const double fl = floor(fc);
                s_i[d][threadIdx.x] = (int)fl;
                s_w[d][threadIdx.x] = fc - fl;
                const double Ub = A.pt[(3 + d) * a.n_act + p];
                s_u[d][threadIdx.x] = ns > 1 ? Ub / (double)ns : Ub;
            }
        }
        __syncthreads();
        for (int s = 0; s < cnt; ++s) {
            const int dx = ci - s_i[0][s], dy = cj - s_i[1][s], dz = ck - s_i[2][s];
            if (dx < 0 || dx > 1 || dy < 0 || dy > 1 || dz < 0 || dz > 1) continue;
            const double w1[3] = {s_w[0][s], s_w[1][s], s_w[2][s]};
            const double w = (dx ? w1[0] : 1.0 - w1[0]) * (dy ? w1[1] : 1.0 - w1[1]) * (dz ? w1[2] : 1.0 - w1[2]);
            double dot = 0.0;
            for (int c = 0; c < 3; ++c) {
                const double Ub = s_u[c][s];
                lam[1 + c] += w * Ub / rho;
                dot += Ub * Uc[c];
            }
            lam[0] += -w * dot / rho;
            touched = true;
        }
    }
    if (ok && touched)
        for (int v = 0; v < 4; ++v) A.lam[v][q] = lam[v];
}

hipError_t launch_alm_adjoint(const AlmAdjArgs& A, hipStream_t s) {
    const int n = A.fwd.n_act;
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(alm_adj_gather_kernel, dim3(n), dim3(256), 0, s, A);
    hipLaunchKernelGGL(alm_adj_points_kernel, dim3((n + 63) / 64), dim3(64), 0, s, A);
    const long long ncell = (long long)A.fwd.samp_n[0] * A.fwd.samp_n[1] * A.fwd.samp_n[2];
    hipLaunchKernelGGL(alm_adj_scatter_kernel, dim3((unsigned)((ncell + 255) / 256)), dim3(256), 0, s, A);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// workspace
// ------------------------------------------------------------------------------------------------
AdjSplit adj_split(int n_n, int n_t1, int n_t2) {
    AdjSplit s;
    s.tiles_t1 = (n_t1 + TILE1 - 1) / TILE1;
    s.tiles_t2 = (n_t2 + AdjTile::T2 - 1) / AdjTile::T2;
    s.chunk = face_chunk(n_n + 1, s.tiles_t1 * s.tiles_t2, ADJ_SLOTS);
    s.nch = (n_n + 1 + s.chunk - 1) / s.chunk;
    s.x1 = std::min(EXT1, n_t1 + 4);
    s.x2 = std::min(AdjTile::T2 + 4, n_t2 + 4);
    return s;
}

void adjoint_carve(char* base, int nx, int ny, int nz, int n_act, AdjBuffers* b, size_t* total) {
    size_t off = 0;
    auto take = [&](size_t bytes) -> char* {
        char* p = base ? base + off : nullptr;
        off += (bytes + 255) & ~size_t(255);
        return p;
    };
    const size_t np = (size_t)(nx + 6) * (ny + 6) * (nz + 6);
    double** pads[4] = {b->lam, b->lam_star, b->lam_new, b->star_t};
    for (int a = 0; a < 4; ++a)
        for (int v = 0; v < 4; ++v) pads[a][v] = reinterpret_cast<double*>(take(np * 8));
    const int n[3] = {nx, ny, nz};
    const int ax[3][3] = {{0, 1, 2}, {1, 0, 2}, {2, 0, 1}};
    size_t cells = 0;  // doubles of the tile kernel's output
    for (int d = 0; d < 3; ++d) {
        const AdjSplit sp = adj_split(n[ax[d][0]], n[ax[d][1]], n[ax[d][2]]);
        cells = std::max(cells, (size_t)sp.tiles_t1 * sp.tiles_t2 * sp.nch * (sp.chunk + 5) * 4 * sp.x1 * sp.x2);
    }
    b->slab = reinterpret_cast<double*>(take(cells * 8));
    b->pt = reinterpret_cast<double*>(take(16 * (size_t)std::max(n_act, 1) * 8));
    *total = off;
}

size_t adjoint_workspace_bytes(int nx, int ny, int nz, int n_act) {
    AdjBuffers b;
    size_t t = 0;
    adjoint_carve(nullptr, nx, ny, nz, n_act, &b, &t);
    return t;
}

}  // namespace gks
