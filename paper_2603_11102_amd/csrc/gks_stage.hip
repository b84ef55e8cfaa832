// gks_stage.hip -- the FP32 S2O4 stage kernels (the FP64 ones are in gks_stage64.hip): reconstruction,
// gas-kinetic flux, flux divergence and the stage combination, the x and y directions in one launch and z in one,
// or all three together on small grids (Section 2,
// Eqs. (semi), (finite), (x_example), (flux); the two-stage fourth-order combinations). Also the work split
// of both precisions.
//
// One workgroup owns a tile of 16 x 16 faces in the tangential plane (512 threads = 8 wave64) and marches
// along the face normal through a chunk of faces (or through an equal share of the tile-major (tile, cell)
// order, one march per tile the share meets, when the tiles do not divide the resident workgroup slots: see
// face_split):
//   * column phase: each of the 20 x 20 tangential columns (tile + 2-cell halo per side) keeps a
//     5-cell window of the field in registers; per cell it evaluates the WENO-JS values at both of its
//     faces with one set of smoothness indicators, the normal derivative D (cubic through four cells)
//     and C = (q^L + q^R)/2 for all four variables -> LDS;
//   * t1 phase: WENO-JS at the two Gauss points of q^L, q^R, quartic Gauss values of D and C and the
//     quartic Gauss derivative of C along t1, the 4 x 320 (variable, position) items spread over all
//     threads -> LDS;
//   * t2 phase: the same along t2 for each Gauss line, giving per Gauss point q^L, q^R, dQ/dn, dQ/dt1,
//     dQ/dt2 in registers (one thread per face and Gauss line);
//   * flux phase: closed-form flux per Gauss point, quadrature over the face, divergence against the
//     previous face of the column, and the accumulation (or the S2O4 epilogue in the last direction).
// No face flux is written to memory. The phases run as a software pipeline over two LDS buffers
// (the face step of f, the t1 phase of f + 1 and the column phase of f + 2 between two barriers; 155 KB of
// the 160 KB per CU).
#include <algorithm>

#include "gks_internal.h"

namespace gks {

template <typename T>
__device__ __forceinline__ T pick(bool c, T x, T y) {
    return c ? x : y;
}

template <typename real>
struct Vec2;
template <>
struct Vec2<float> {
    using type = float2;
};
// The pair of variables (2m, 2m + 1) of cell i in an array that holds four variables per cell.
template <typename real>
__device__ __forceinline__ typename Vec2<real>::type ld2(const real* p, long long i, int m) {
    return *reinterpret_cast<const typename Vec2<real>::type*>(p + 4 * i + 2 * m);
}
template <typename real>
__device__ __forceinline__ void st2(real* p, long long i, int m, typename Vec2<real>::type v) {
    *reinterpret_cast<typename Vec2<real>::type*>(p + 4 * i + 2 * m) = v;
}

// The value of the partner lane (lane ^ 1; all lanes are active where it is used), moved through the LDS
// crossbar (ds_bpermute), off the VALU that bounds the kernel.
__device__ __forceinline__ float pair_swap(float x) { return __shfl_xor(x, 1); }

// LDS: two buffers, so that the phases of consecutive faces overlap; per variable the column values
// [q^L, q^R, D, C][t2 row][t1 column] and the t1-phase results
// [q^L_m, q^R_m, D_m, (dC/dt1)_m, C_m][t2 row][t1 position][Gauss line m]. A wave of the t1 phase takes
// one row of all four variables, 16 consecutive positions each; the variable blocks are padded to
// start 16 words apart modulo 64, so its reads meet no bank twice, and the t1-phase results of the four
// variables start 32 words apart modulo 64, the least the wave's 64-bit stores can share banks.
struct FaceLds {
    struct {
        float a[4][EXT2][EXT1];
        float pad[16];
    } nrm[2][4];
    struct {
        float a[5][EXT2][TILE1][2];
        float pad[32];
    } t1[2][4];
    float range[2][FACE_THREADS / 64];
};

// The marches of workgroup blk of the nblk (a multiple of 8) that take this direction.
// MODE (the direction's role): 3 = x pass, writes its residual to the blocked arrays; 0 = y pass,
// writes the main residual arrays; 4 = z pass, adds both and applies the S2O4 stage update; 5 = z pass
// beside the other two, leaves its residual where the stage update will stand (combine_kernel does it).
// STR: the mesh is stretched and the spacings come from the per-axis arrays; otherwise the uniform
// inverse spacings are kernel arguments (no memory access for them inside the march).
template <typename real, int STAGE, int MODE, bool STR>
__device__ __forceinline__ void face_march(const FaceArgs<real>& a, const int blk, const int nblk, FaceLds& lds) {
    static_assert(MODE == 0 || MODE == 3 || MODE == 4 || MODE == 5, "face pass mode");
    // TILE1 x T2 faces, EXT1 x X2 columns, NTH threads
    constexpr int T2 = TILE2, X2 = EXT2, NTH = FACE_THREADS;
    static_assert(EXT1 * X2 <= NTH && 2 * TILE1 * T2 == NTH, "one thread per column and per face line");
    constexpr bool NEED_F0 = (STAGE == 1);
    using real2 = typename Vec2<real>::type;
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
    // one march per tile the range meets (the shift cm, the window and the face fluxes restart)
    while (lin < lin_end) {
    const int tile = (int)(lin / a.n_n);
    const int f0 = (int)(lin - (long long)tile * a.n_n);
    const int f1 = (int)min((long long)a.n_n, f0 + (lin_end - lin));  // residuals of cells [f0, f1); faces f0..f1
    lin += f1 - f0;
    const int tile1 = tile % a.tiles_t1, tile2 = tile / a.tiles_t1;
    const int j0 = tile1 * TILE1, k0 = tile2 * T2;
    const real eps = a.eps;

    // column role
    const bool col = tid < EXT1 * X2;
    const int c1 = tid % EXT1, c2 = tid / EXT1;
    const int jc = j0 - 2 + c1, kc = k0 - 2 + c2;
    const bool col_ld = col && (jc < a.n_t1 + NG) && (kc < a.n_t2 + NG);
    const long long cbase = a.pad0 + (long long)jc * a.st_t1 + (long long)kc * a.st_t2;
    // the in-loop prefetch of the column cells is done by every thread, columns outside the padded domain
    // and threads without a column reading a clamped column (its values are never used): a load on every
    // path leaves the compiler no merge of a loaded and a kept value, which would make it wait for the
    // load within the same step, and for the step's stores at the next one
    const long long cbase_ld = a.pad0 + (long long)min(jc, a.n_t1 + NG - 1) * a.st_t1 +
                               (long long)min(k0 - 2 + min(c2, X2 - 1), a.n_t2 + NG - 1) * a.st_t2;
    // face role: face (fj, fk) of the tile, Gauss line m (partner lane tid ^ 1 holds the other line)
    const int m = tid & 1;
    const int fj = (tid >> 1) % TILE1, fk = (tid >> 1) / TILE1;
    const bool face_ok = (j0 + fj < a.n_t1) && (k0 + fk < a.n_t2);

    // Inside the kernel the normal momentum is carried as its deviation from a workgroup constant
    // cm (the midrange of its values in the first window of the tile), so that the O(1) part of the
    // mass flux cancels exactly between the two faces of a cell and FP32 rounding acts on the deviation
    // only. The WENO and linear stencils commute with the shift (their weights sum to one and the
    // smoothness indicators use differences); the derivatives are unchanged.
    real cm;
    real ring[4][5];
    real carry[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        carry[v] = real(0);
#pragma unroll
        for (int r = 0; r < 5; ++r) ring[v][r] = real(0);
    }
    // warm-up: window of cells f0-3 .. f0+1, then the right-face value of cell f0-1 (q^L of face f0)
    if (col_ld) {
#pragma unroll
        for (int r = 0; r < 5; ++r) {
            const long long idx = cbase + (long long)(f0 - 3 + r) * a.st_n;
#pragma unroll
            for (int v = 0; v < 4; ++v) ring[v][r] = a.q[v][idx];
        }
    }
    {
        auto& s_range = lds.range;
        float lo = col_ld ? float(ring[1][0]) : 3.0e38f, up = col_ld ? float(ring[1][0]) : -3.0e38f;
#pragma unroll
        for (int r = 1; r < 5; ++r) {
            lo = col_ld ? fminf(lo, float(ring[1][r])) : lo;
            up = col_ld ? fmaxf(up, float(ring[1][r])) : up;
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            lo = fminf(lo, __shfl_xor(lo, o));
            up = fmaxf(up, __shfl_xor(up, o));
        }
        if ((tid & 63) == 0) {
            s_range[0][tid >> 6] = lo;
            s_range[1][tid >> 6] = up;
        }
        __syncthreads();
        lo = s_range[0][0];
        up = s_range[1][0];
#pragma unroll
        for (int w = 1; w < NTH / 64; ++w) {
            lo = fminf(lo, s_range[0][w]);
            up = fmaxf(up, s_range[1][w]);
        }
        cm = lo <= up ? real(0.5f * (lo + up)) : real(0);
#pragma unroll
        for (int r = 0; r < 5; ++r) ring[1][r] -= cm;
    }
    if (col_ld) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            real right, left;
            weno_faces<real>(ring[v][0], ring[v][1], ring[v][2], ring[v][3], ring[v][4], eps, right, left);
            carry[v] = right;
        }
    }
    // software pipelining: the cell entering the window at the next step is loaded one step ahead
    real nxt[4] = {real(0), real(0), real(0), real(0)};
    if (col_ld) {
        const long long idx = cbase + (long long)(f0 + 2) * a.st_n;
#pragma unroll
        for (int v = 0; v < 4; ++v) nxt[v] = a.q[v][idx];
    }
    const real dt = real(*a.dt_ptr);
    // the previous face's fluxes of this lane's two variables
    real2 pprev0 = {0, 0}, pprev1 = {0, 0};

    const bool hi = m != 0;
    // tangential inverse widths, loaded once (a vector load inside the march would make the wait for
    // it also wait for the column prefetch): t2 of this thread's face line, as scaled coefficients (in the t1
    // phase these cost more registers than they save: z pass 4 -> 11 spilled, 0.6 % slower); t1 of its t1-phase
    // items, whose t1 position is tid % TILE1 for every item
    const QuarticDeriv<real> qd2(STR ? a.ih2[min(k0 + fk, a.n_t2 - 1)] : a.inv_h2);
    const real ih1 = STR ? a.ih1[min(j0 + tid % TILE1, a.n_t1 - 1)] : a.inv_h1;
    // epilogue operands (z pass) of cell f - 1
    struct Epi {
        real2 r0, r1, x0, x1, lo;
        real q[2];
    };
    auto epi_load = [&](int f, Epi& ep) {
        if constexpr (MODE == 4) {
            // loaded on every path (for the same reason as the column prefetch): at f = f0, one face past
            // the march and for faces outside the domain a clamped cell is read and its values are not used
            const int cell = min(max(f - 1, 0), a.n_n - 1), je = min(j0 + fj, a.n_t1 - 1), ke = min(k0 + fk, a.n_t2 - 1);
            const long long ridx = (long long)cell * a.ist_n + (long long)je * a.ist_t1 + (long long)ke * a.ist_t2;
            const long long pidx = a.pad0 + (long long)cell * a.st_n + (long long)je * a.st_t1 + (long long)ke * a.st_t2;
            const long long xidx = rx_block_index(je, ke, cell, a.rx_nx, a.rx_nyb);
            ep.r1 = ld2(a.r1, ridx, m);
            ep.x1 = ld2(a.rx1, xidx, m);
            ep.lo = ld2(a.lo_in, ridx, m);
            if (NEED_F0) {
                ep.r0 = ld2(a.r0, ridx, m);
                ep.x0 = ld2(a.rx0, xidx, m);
            }
#pragma unroll
            for (int vv = 0; vv < 2; ++vv) {
                const real* const src = NEED_F0 ? pick(hi, a.q_c[LOC[2 + vv]], a.q_c[LOC[vv]])
                                                : pick(hi, a.s_in[LOC[2 + vv]], a.s_in[LOC[vv]]);
                ep.q[vv] = src[pidx];
            }
        }
    };
    // column phase of face f into LDS buffer buf
    auto column_step = [&](int f, int buf) {
        const real ihf_f = STR ? a.ihf[f] : a.inv_hn;  // inverse spacing at face f (normal derivative)
        // ---- column phase (all variables): window cells f-2 .. f+2, prefetch cell f+3
        if (col) {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
#pragma unroll
                for (int r = 0; r < 4; ++r) ring[v][r] = ring[v][r + 1];
                // the shift is applied here, a step after the load, so that the prefetch stays in flight
                ring[v][4] = v == 1 ? nxt[v] - cm : nxt[v];
            }
        }
        {
            const long long idx = cbase_ld + (long long)min(f + 3, a.n_n + 2) * a.st_n;
#pragma unroll
            for (int v = 0; v < 4; ++v) nxt[v] = a.q[v][idx];
        }
        if (col) {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                real right, left;
                weno_faces<real>(ring[v][0], ring[v][1], ring[v][2], ring[v][3], ring[v][4], eps, right, left);
                const real qL = carry[v];
                const real D = (ring[v][0] - real(15) * ring[v][1] + real(15) * ring[v][2] - ring[v][3]) *
                               (real(1.0 / 12.0) * ihf_f);
                s_nrm[buf][v].a[0][c2][c1] = qL;
                s_nrm[buf][v].a[1][c2][c1] = left;
                s_nrm[buf][v].a[2][c2][c1] = D;
                s_nrm[buf][v].a[3][c2][c1] = real(0.5) * (qL + left);
                carry[v] = right;
            }
        }
    };
    // t1 phase of LDS buffer buf
    auto t1_step = [&](int buf) {
        // ---- t1 phase: the 4 x 16 x X2 items (variable v, t2 row tk, t1 position tj) spread over all
        // threads in row-wave order: a thread keeps tj = tid % 16 and v = tid / 16 % 4 and takes the rows
        // tid / 64 + k NTH / 64, so its LDS addresses move by a fixed step (no index arithmetic in the
        // march)
        static_assert(TILE1 == 16 && NTH % 64 == 0, "t1 items: 16 positions x 4 variables per wave");
        {
            constexpr int RSTEP = NTH / 64, NK = (X2 + RSTEP - 1) / RSTEP;
            const int tj = tid & 15, v = (tid >> 4) & 3;
#pragma unroll
            for (int kk = 0; kk < NK; ++kk) {
                const int tk = (tid >> 6) + kk * RSTEP;
                if (X2 % RSTEP == 0 || tk < X2) {
                    real x[4][5];
#pragma unroll
                    for (int q = 0; q < 4; ++q)
#pragma unroll
                        for (int r = 0; r < 5; ++r) x[q][r] = s_nrm[buf][v].a[q][tk][tj + r];
                    real vm, vp;
                    weno_gauss<real>(x[0][0], x[0][1], x[0][2], x[0][3], x[0][4], eps, vm, vp);
                    s_t1[buf][v].a[0][tk][tj][0] = vm;
                    s_t1[buf][v].a[0][tk][tj][1] = vp;
                    weno_gauss<real>(x[1][0], x[1][1], x[1][2], x[1][3], x[1][4], eps, vm, vp);
                    s_t1[buf][v].a[1][tk][tj][0] = vm;
                    s_t1[buf][v].a[1][tk][tj][1] = vp;
                    quartic_gauss_value<real>(x[2][0], x[2][1], x[2][2], x[2][3], x[2][4], vm, vp);
                    s_t1[buf][v].a[2][tk][tj][0] = vm;
                    s_t1[buf][v].a[2][tk][tj][1] = vp;
                    quartic_gauss_deriv<real>(x[3][0], x[3][1], x[3][2], x[3][3], x[3][4], vm, vp);
                    s_t1[buf][v].a[3][tk][tj][0] = vm * ih1;
                    s_t1[buf][v].a[3][tk][tj][1] = vp * ih1;
                    quartic_gauss_value<real>(x[3][0], x[3][1], x[3][2], x[3][3], x[3][4], vm, vp);
                    s_t1[buf][v].a[4][tk][tj][0] = vm;
                    s_t1[buf][v].a[4][tk][tj][1] = vp;
                }
            }
        }
    };
    // t2 phase, flux and residual (or stage update) of face f from LDS buffer buf
    auto face_step = [&](int f, int buf, const Epi& ep) {
        // ---- t2 phase: per thread one face and one Gauss line, all variables
        real gp[4][2][5];  // [variable][Gauss n][q^L, q^R, d/dn, d/dt1, d/dt2]
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            real y[5][5];
#pragma unroll
            for (int q = 0; q < 5; ++q)
#pragma unroll
                for (int r = 0; r < 5; ++r) y[q][r] = s_t1[buf][v].a[q][fk + r][fj][m];
            real vm, vp;
            weno_gauss<real>(y[0][0], y[0][1], y[0][2], y[0][3], y[0][4], eps, vm, vp);
            gp[v][0][0] = vm;
            gp[v][1][0] = vp;
            weno_gauss<real>(y[1][0], y[1][1], y[1][2], y[1][3], y[1][4], eps, vm, vp);
            gp[v][0][1] = vm;
            gp[v][1][1] = vp;
            quartic_gauss_value<real>(y[2][0], y[2][1], y[2][2], y[2][3], y[2][4], vm, vp);
            gp[v][0][2] = vm;
            gp[v][1][2] = vp;
            quartic_gauss_value<real>(y[3][0], y[3][1], y[3][2], y[3][3], y[3][4], vm, vp);
            gp[v][0][3] = vm;
            gp[v][1][3] = vp;
            qd2(y[4][0], y[4][1], y[4][2], y[4][3], y[4][4], vm, vp);
            gp[v][0][4] = vm;
            gp[v][1][4] = vp;
        }

        // ---- flux at this thread's two Gauss points (their quadrature weight 1/4 is part of the divergence)
        real fa0[4], fa1[4];
#pragma unroll
        for (int n = 0; n < 2; ++n) {
            real qL[4], qR[4], g[3][4], f0n[4], f1n[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                qL[v] = gp[v][n][0];
                qR[v] = gp[v][n][1];
                g[0][v] = gp[v][n][2];
                g[1][v] = gp[v][n][3];
                g[2][v] = gp[v][n][4];
            }
            gp_flux<real, NEED_F0, true>(qL, qR, g, a.fc, f0n, f1n, cm);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                fa1[v] = n == 0 ? f1n[v] : fa1[v] + f1n[v];
                if (NEED_F0) fa0[v] = n == 0 ? f0n[v] : fa0[v] + f0n[v];
            }
        }
        // sum with the partner lane, scattered: lane m keeps the global variables 2m and 2m + 1 (local indices
        // LOC[2m], LOC[2m + 1]) and sends the other two, picked by value with a per-lane select between
        // compile-time indices (indexing a register array with the lane-dependent index would move it to scratch).
        // Against all four sums in both lanes, with the selects after them: 12 of 456 instructions and 10 registers
        // less (192x96x96, with the scaled t2 coefficients: 2.0 % of the step).
        auto pair_sum = [&](const real (&x)[4]) -> real2 {
            real2 r;
            r.x = pick(hi, x[LOC[2]], x[LOC[0]]) + pair_swap(pick(hi, x[LOC[0]], x[LOC[2]]));
            r.y = pick(hi, x[LOC[3]], x[LOC[1]]) + pair_swap(pick(hi, x[LOC[1]], x[LOC[3]]));
            return r;
        };
        const real2 fcur1 = pair_sum(fa1);
        const real2 fcur0 = NEED_F0 ? pair_sum(fa0) : real2{0, 0};
        if (f > f0 && face_ok) {
            const int cell = f - 1;
            const long long ridx = (long long)cell * a.ist_n + (long long)(j0 + fj) * a.ist_t1 +
                                   (long long)(k0 + fk) * a.ist_t2;
            const long long pidx = a.pad0 + (long long)cell * a.st_n + (long long)(j0 + fj) * a.st_t1 +
                                   (long long)(k0 + fk) * a.st_t2;
            // lane m owns the global variables 2m and 2m + 1 (local indices LOC[2m], LOC[2m + 1]); the
            // residual and low-order arrays hold the four variables of a cell together, so the lane moves
            // them as one pair. Per-variable pointers and values are picked by value with a per-lane select
            // between compile-time indices: indexing the argument or register arrays with the
            // lane-dependent index would fetch pointers from memory and move the arrays to scratch.
            real2 d1, d0;
            const real ihc = real(0.25) * (STR ? a.ihc[cell] : a.inv_hn);  // 1/4: weight of a Gauss point
            d1.x = (pprev1.x - fcur1.x) * ihc;
            d1.y = (pprev1.y - fcur1.y) * ihc;
            if (NEED_F0) {
                d0.x = (pprev0.x - fcur0.x) * ihc;
                d0.y = (pprev0.y - fcur0.y) * ihc;
            } else {
                d0.x = d0.y = real(0);
            }
            if constexpr (MODE == 3) {
                const long long xidx = rx_block_index(cell, j0 + fj, k0 + fk, a.rx_nx, a.rx_nyb);
                st2(a.rx1, xidx, m, d1);
                if (NEED_F0) st2(a.rx0, xidx, m, d0);
            } else if constexpr (MODE == 0) {
                st2(a.r1, ridx, m, d1);
                if (NEED_F0) st2(a.r0, ridx, m, d0);
            } else if constexpr (MODE == 5) {
                pick(hi, a.out_a[LOC[2]], a.out_a[LOC[0]])[pidx] = d1.x;
                pick(hi, a.out_a[LOC[3]], a.out_a[LOC[1]])[pidx] = d1.y;
                if (NEED_F0) {
                    pick(hi, a.out_b[LOC[2]], a.out_b[LOC[0]])[pidx] = d0.x;
                    pick(hi, a.out_b[LOC[3]], a.out_b[LOC[1]])[pidx] = d0.y;
                }
            } else {
                const real2 r1v = ep.r1, x1v = ep.x1, r0v = ep.r0, x0v = ep.x0;
                const real L1[2] = {r1v.x + (d1.x + x1v.x), r1v.y + (d1.y + x1v.y)};
                const real L0[2] = {r0v.x + (d0.x + x0v.x), r0v.y + (d0.y + x0v.y)};
                // the state is carried as hi + lo; each update is an error-free sum of the
                // stored high part and (low part + increment)
                const real lo[2] = {ep.lo.x, ep.lo.y};
                real2 la = {0, 0}, lb = {0, 0};
#pragma unroll
                for (int vv = 0; vv < 2; ++vv) {
                    real* const outa = pick(hi, a.out_a[LOC[2 + vv]], a.out_a[LOC[vv]]);
                    float sh, sl;
                    if (NEED_F0) {
                        real* const outb = pick(hi, a.out_b[LOC[2 + vv]], a.out_b[LOC[vv]]);
                        two_sum(ep.q[vv], lo[vv] + (real(0.5) * dt * L0[vv] + real(0.125) * dt * dt * L1[vv]), sh, sl);
                        outa[pidx] = sh;
                        if (vv == 0) la.x = sl; else la.y = sl;
                        two_sum(ep.q[vv], lo[vv] + (dt * L0[vv] + (dt * dt * real(1.0 / 6.0)) * L1[vv]), sh, sl);
                        outb[pidx] = sh;
                        if (vv == 0) lb.x = sl; else lb.y = sl;
                    } else {
                        // body force G on the momenta (global variables 1..3)
                        const real gv = pick(hi, a.g_global[1 + vv], vv == 1 ? a.g_global[0] : real(0));
                        const real add = (dt * dt * real(1.0 / 3.0)) * L1[vv] + dt * gv;
                        two_sum(ep.q[vv], lo[vv] + add, sh, sl);
                        outa[pidx] = sh;
                        if (vv == 0) la.x = sl; else la.y = sl;
                    }
                }
                st2(a.lo_a, ridx, m, la);
                if (NEED_F0) st2(a.lo_b, ridx, m, lb);
            }
        }
        pprev1 = fcur1;
        if (NEED_F0) pprev0 = fcur0;
    };
    // software pipeline over two LDS buffers with one barrier per face: the face step of f reads
    // s_t1[buf], the t1 phase of f + 1 reads s_nrm[buf ^ 1] and writes s_t1[buf ^ 1], the column
    // phase of f + 2 writes s_nrm[buf]; each buffer was last read or written before the previous
    // barrier. The epilogue operands of the next face step are loaded one step ahead. Waves whose
    // column phase is light (400 columns on 512 threads) go on to the next face's work.
    Epi ep = {};
    epi_load(f0, ep);
    column_step(f0, 0);
    __syncthreads();
    t1_step(0);
    column_step(f0 + 1, 1);
    __syncthreads();
    for (int f = f0; f <= f1; ++f) {
        const int buf = (f - f0) & 1;
        face_step(f, buf, ep);
        epi_load(f + 1, ep);
        if (f + 1 <= f1) t1_step(buf ^ 1);
        if (f + 2 <= f1) column_step(f + 2, buf);
        __syncthreads();
    }
    }  // segments
}

// x and y passes in one launch: the workgroups of both directions share the chip, so a workgroup marches twice
// as far as in a launch of its own and the start of a march (about 1.5 face steps) and the launch's end
// are paid once.
template <typename real, int STAGE, bool STR>
__global__ void __launch_bounds__(FACE_THREADS) face_xy_kernel(const FaceArgs<real> ax, const FaceArgs<real> ay) {
    __shared__ FaceLds lds;
    const int nx = pad8(ax.n_wg), blk = blockIdx.x;
    if (blk < nx) face_march<real, STAGE, 3, STR>(ax, blk, nx, lds);
    else face_march<real, STAGE, 0, STR>(ay, blk - nx, pad8(ay.n_wg), lds);
}

// the z pass with the stage update
template <typename real, int STAGE, bool STR>
__global__ void __launch_bounds__(FACE_THREADS) face_z_kernel(const FaceArgs<real> a) {
    __shared__ FaceLds lds;
    if (STAGE == 2 && a.finish && blockIdx.x == 0 && threadIdx.x == 0) finish_step(a.finish);
    face_march<real, STAGE, 4, STR>(a, blockIdx.x, pad8(a.n_wg), lds);
}

// all three directions in one launch, for grids that leave much of the chip idle in each (combine_kernel follows)
template <typename real, int STAGE, bool STR>
__global__ void __launch_bounds__(FACE_THREADS) face_xyz_kernel(const FaceArgs<real> ax, const FaceArgs<real> ay,
                                                                const FaceArgs<real> az, const DtArgs dt) {
    __shared__ FaceLds lds;
    const int nx = pad8(ax.n_wg), ny = pad8(ay.n_wg), blk = blockIdx.x;
    if (STAGE == 1 && blk == (int)gridDim.x - 1) {
        // one more workgroup forms the time step, which the stage update is the first to read
        static_assert(sizeof(lds.nrm) >= sizeof(double) * (FACE_THREADS / 64), "LDS of dt_update");
        dt_update<FACE_THREADS>(dt, reinterpret_cast<double*>(&lds.nrm));
        return;
    }
    if (blk < nx) face_march<real, STAGE, 3, STR>(ax, blk, nx, lds);
    else if (blk < nx + ny) face_march<real, STAGE, 0, STR>(ay, blk - nx, ny, lds);
    else face_march<real, STAGE, 5, STR>(az, blk - nx - ny, pad8(az.n_wg), lds);
}

template <>
int face_slots<float>(int) {
    // workgroups of the face kernels that the device holds at once
    int dev = 0, cus = 0, per_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, face_z_kernel<float, 1, false>, FACE_THREADS, 0) !=
        hipSuccess)
        return 0;
    return cus * per_cu;
}

int face_chunk(int n_n, int tiles, int slots) {
    // Workgroups of one launch run in rounds of `slots`; a workgroup costs about (chunk + 2) face steps
    // (chunk + 1 faces, and the column phase primes five planes before the first one). Pick the chunk
    // that minimises rounds x (chunk + 2); ties go to the longer chunk.
    if (slots <= 0) slots = 512;
    int best_chunk = n_n;
    long long best = -1;
    for (int nc = 1; nc <= n_n; ++nc) {
        const int chunk = (n_n + nc - 1) / nc;
        const long long wgs = (long long)tiles * ((n_n + chunk - 1) / chunk);
        const long long cost = ((wgs + slots - 1) / slots) * (chunk + 2);
        if (best < 0 || cost < best) {
            best = cost;
            best_chunk = chunk;
        }
    }
    return best_chunk;
}

int face_split(const FaceDir* dirs, int ndirs, int slots, FaceSplit* out) {
    // The least T, in face steps, at which the directions' workgroups of at most T steps each fit the `slots`
    // that run at once (a march over L cells costs about L + 2). Per direction either aligned chunks of T - 2
    // cells, or equal runs of the tile-major (tile, cell) order, which fill the slots when the tiles do not
    // divide them but pay two steps more where a run crosses into the next tile; the fewer workgroups win.
    // Counts are rounded up to a multiple of 8 per direction: workgroups go round-robin to the 8 XCDs, and a
    // rest that piles up on the first ones gives those a second round (the 192 x 96 x 96 channel in one
    // launch took 1.9 times as long).
    if (slots <= 0) slots = 512;
    auto fewest = [&](const FaceDir& d, int T, FaceSplit* o) {
        const long long total = (long long)d.tiles * d.n;
        const int chunk = std::min(T - 2, d.n);
        long long best = (long long)d.tiles * ((d.n + chunk - 1) / chunk);
        o->seg_len = 0;
        o->chunk = chunk;
        // A run of len cells at offset off in its tile takes len + 2 (tiles it meets) steps. Fewer than `first` tiles are
        // fewer than any run of T - 2 segs cells meets (unless one run is everything), and runs only get shorter and
        // more with segs: the first length that fits is the one sought, at most two steps on.
        const int first = total <= T - 2 ? 1 : (T - 1) / (d.n + 2) + 1;
        for (int segs = first; segs <= (T - 2) / d.n + 2; ++segs) {
            const long long len = std::min((long long)T - 2 * segs, total);
            if (len < 1) break;
            const long long wgs = (total + len - 1) / len;
            if (wgs >= best || wgs > slots) break;
            const long long met = (len - 1) / d.n + 1, rem = (len - 1) % d.n;  // tiles met from off = 0; met + 1 if off + rem >= n
            if (len + 2 * met > T) continue;
            bool fits = true;
            if (len + 2 * (met + 1) > T) {
                long long off = 0;
                for (long long w = 0; fits && w < wgs; ++w) {
                    const long long l = std::min(len, total - w * len);
                    fits = l == len ? off + rem < d.n : l + 2 * ((off + l - 1) / d.n + 1) <= T;
                    off += rem + 1;
                    if (off >= d.n) off -= d.n;
                }
            }
            if (!fits) continue;
            best = wgs;
            o->seg_len = (int)len;
            break;
        }
        o->n_wg = best;
        return best;
    };
    auto total_wgs = [&](int T, FaceSplit* o) {
        long long n = 0;
        for (int d = 0; d < ndirs; ++d) n += (fewest(dirs[d], T, o + d) + 7) / 8 * 8;
        return n;
    };
    int lo = 3, hi = 3;
    while (total_wgs(hi, out) > slots && hi < (1 << 29)) {
        lo = hi + 1;
        hi *= 2;
    }
    while (lo < hi) {
        const int mid = lo + (hi - lo) / 2;
        if (total_wgs(mid, out) <= slots) hi = mid;
        else lo = mid + 1;
    }
    total_wgs(hi, out);
    return hi;
}

FacePlan face_plan(const int n[3], bool f64, const int slots[2]) {
    // Each tile height (FP64: two, see FACE64_ROWS) in both launch schemes, by estimated time in ns: face steps
    // of the longest workgroup times the step, and per launch its start and end.
    constexpr int ax[3][3] = {{0, 1, 2}, {1, 0, 2}, {2, 0, 1}};  // (normal, t1, t2)
    const double cells = (double)n[0] * n[1] * n[2];
    double best = -1.0;
    FacePlan plan{};
    for (int o = 0; o < (f64 ? 2 : 1); ++o) {
        const int rows = f64 ? FACE64_ROWS[o] : TILE2;
        const double step = f64 ? FACE64_STEP[o] : FACE32_STEP;
        FaceDir dir[3];
        for (int d = 0; d < 3; ++d)
            dir[d] = FaceDir{n[ax[d][0]], ((n[ax[d][1]] + TILE1 - 1) / TILE1) * ((n[ax[d][2]] + rows - 1) / rows)};
        for (int scheme = 0; scheme < 2; ++scheme) {
            FaceSplit sp[3];
            double t;
            if (scheme == 0) {
                t = step * (face_split(dir, 2, slots[o], sp) + face_split(dir + 2, 1, slots[o], sp + 2)) + 2 * FACE_LAUNCH;
            } else {
                // eight slots are left to the workgroup that forms the time step
                t = step * face_split(dir, 3, slots[o] - 8, sp) + FACE_LAUNCH + COMBINE_LAUNCH +
                    (f64 ? COMBINE_CELL64 : COMBINE_CELL32) * cells;
            }
            if (best < 0.0 || t < best) {
                best = t;
                plan.side_by_side = scheme;
                plan.rows = rows;
                for (int d = 0; d < 3; ++d) {
                    plan.chunk[d] = sp[d].chunk;
                    plan.seg_len[d] = sp[d].seg_len;
                    plan.n_wg[d] = (int)sp[d].n_wg;
                }
            }
        }
    }
    return plan;
}

#define GKS_LAUNCH_STR(KERNEL, ST, BLOCKS, ...)                                                               \
    do {                                                                                                      \
        const dim3 grid((unsigned)(BLOCKS)), block(FACE_THREADS);                                             \
        if (str) hipLaunchKernelGGL((KERNEL<float, ST, true>), grid, block, 0, s, __VA_ARGS__);               \
        else hipLaunchKernelGGL((KERNEL<float, ST, false>), grid, block, 0, s, __VA_ARGS__);                  \
        return hipGetLastError();                                                                             \
    } while (0)

template <>
hipError_t launch_face_xy<float>(const FaceArgs<float>& ax, const FaceArgs<float>& ay, int stage, hipStream_t s) {
    const bool str = ax.stretched != 0;
    const long long blocks = (long long)pad8(ax.n_wg) + pad8(ay.n_wg);
    if (stage == 1) GKS_LAUNCH_STR(face_xy_kernel, 1, blocks, ax, ay);
    else GKS_LAUNCH_STR(face_xy_kernel, 2, blocks, ax, ay);
}

template <>
hipError_t launch_face_z<float>(const FaceArgs<float>& a, int stage, hipStream_t s) {
    const bool str = a.stretched != 0;
    if (stage == 1) GKS_LAUNCH_STR(face_z_kernel, 1, pad8(a.n_wg), a);
    else GKS_LAUNCH_STR(face_z_kernel, 2, pad8(a.n_wg), a);
}

template <>
hipError_t launch_face_xyz<float>(const FaceArgs<float>& ax, const FaceArgs<float>& ay, const FaceArgs<float>& az,
                                  const DtArgs& dt, int stage, hipStream_t s) {
    const bool str = ax.stretched != 0;
    const long long blocks = (long long)pad8(ax.n_wg) + pad8(ay.n_wg) + pad8(az.n_wg);
    if (stage == 1) GKS_LAUNCH_STR(face_xyz_kernel, 1, blocks + 1, ax, ay, az, dt);
    else GKS_LAUNCH_STR(face_xyz_kernel, 2, blocks, ax, ay, az, dt);
}

}  // namespace gks
