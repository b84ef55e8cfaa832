// gks_device.h -- device math of the high-order isothermal GKS step (gfx950).
//
// Reconstruction (Section 2: fifth-order WENO-JS, dimension by dimension, to the 2x2 Gauss points of
// each face) and the gas-kinetic flux of the interface distribution f = g0 (1 - tau (a.u + A) + A t)
// (Section 2, Eq. (flux); coefficients from the moment system of the Appendix).
//
// Cells have unit width in the stencil formulas; derivatives are scaled by 1/h by the caller.
// Gauss points of a cell are xi = s sqrt(3)/6, s = -1 (m = 0) and s = +1 (m = 1).
//
// Flux: for the isothermal Maxwellian g0 with macroscopic state Q0 and spatial derivatives dQ0/dx_k,
// the moments of f reduce exactly (the Chapman-Enskog identities of the BGK model) to
//   F0 = E_n(Q0) - mu (dU/dx_n + grad U_n)            (no viscous mass flux, no bulk term),
//   F1 = J_n(Q0) Qdot,  Qdot = -sum_k J_k(Q0) dQ0/dx_k  (rho0 <u_n A psi> with A from compatibility),
// where E_k is the isothermal Euler flux and J_k its Jacobian; tau p0 = mu. The constant reference
// pressure c^2 rho_ref is dropped from E_n: it is the same at every face and cancels in the divergence,
// which keeps the O(Ma^2) pressure differences in FP32.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>

namespace gks {

template <typename real> struct Rc;
template <> struct Rc<float> {
    static __device__ __forceinline__ float erf_(float x) { return erff(x); }
    static __device__ __forceinline__ float exp_(float x) { return expf(x); }
    static __device__ __forceinline__ float expm1_(float x) { return expm1f(x); }
};
template <> struct Rc<double> {
    static __device__ __forceinline__ double erf_(double x) { return erf(x); }
    static __device__ __forceinline__ double exp_(double x) { return exp(x); }
    static __device__ __forceinline__ double expm1_(double x) { return expm1(x); }
};

#define GKS_SQRT3 1.7320508075688772935274463415059

// Reciprocal: FP32 uses the hardware v_rcp_f32 (about 1 ulp); FP64 refines v_rcp_f64 (relative error e up
// to 2^-24.4, measured over 2^20 arguments) by the three terms 1 + e + e^2 of its series: error e^3 and about
// 1 ulp of rounding, with one multiply-add less than two Newton steps. Arguments are positive normal numbers here (densities, WENO denominators).
template <typename real> __device__ __forceinline__ real rcp(real x);
template <> __device__ __forceinline__ float rcp<float>(float x) { return __builtin_amdgcn_rcpf(x); }
template <> __device__ __forceinline__ double rcp<double>(double x) {
    const double y = __builtin_amdgcn_rcp(x);
    const double e = fma(-x, y, 1.0);
    return fma(fma(e, e, e), y, y);
}

// a b + c with a wave-uniform c. FP64: v_fma_f64 with c in scalar registers (the compiler's own choice, the
// two-operand v_fmac_f64, first copies c to vector registers: an instruction more).
__device__ __forceinline__ float fma_uniform(float a, float b, float c) { return fmaf(a, b, c); }
__device__ __forceinline__ double fma_uniform(double a, double b, double c) {
    double r;
    asm("v_fma_f64 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "s"(c));
    return r;
}

// Error-free sum (Knuth): s + e == a + b exactly, s = fl(a + b).
__device__ __forceinline__ void two_sum(float a, float b, float& s, float& e) {
    s = a + b;
    const float bb = s - a;
    e = (a - (s - bb)) + (b - bb);
}

// DPP moves inside a row of 16 lanes. In the FP64 face kernels lane bit 2 is h, bit 3 is m; a bank mask picks the four-lane
// banks that take the moved value (the others keep `old`), so a move with a per-lane choice is one instruction per
// word. ZERO: lanes whose source lies outside the row take zero, else they keep `old`.
constexpr int ROW_SHL4 = 0x104, ROW_SHR4 = 0x114, ROW_ROR8 = 0x128;  // from lane + 4, lane - 4, lane ^ 8
constexpr int BANK_H0 = 0x5, BANK_H1 = 0xA, BANK_M0 = 0x3, BANK_M1 = 0xC;

template <int CTRL, int BANK, bool ZERO = false>
__device__ __forceinline__ double dpp_move(double old, double x) {
    const unsigned long long b = (unsigned long long)__double_as_longlong(x);
    const unsigned long long o = (unsigned long long)__double_as_longlong(old);
    const int lo = __builtin_amdgcn_update_dpp((int)(unsigned)(o & 0xffffffffu), (int)(unsigned)(b & 0xffffffffu), CTRL,
                                               0xF, BANK, ZERO);
    const int hi = __builtin_amdgcn_update_dpp((int)(unsigned)(o >> 32), (int)(unsigned)(b >> 32), CTRL, 0xF, BANK, ZERO);
    return __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
}

// ---------------------------------------------------------------------------------------------
// WENO-JS on five cells q[-2..2], written in the stencil's first differences
// d1 = q[-1] - q[-2], d2 = q[0] - q[-1], d3 = q[1] - q[0], d4 = q[2] - q[1]. Sub-stencil k's quadratic
// (cells k-2..k) has second difference a_k and twice its slope at the cell centre b_k (unit cells):
//   a0 = d2 - d1, b0 = 3 d2 - d1;   a1 = d3 - d2, b1 = d2 + d3;   a2 = d4 - d3, b2 = 3 d3 - d4,
// so that its smoothness indicator is 4 beta_k = (13/3) a_k^2 + b_k^2, its values at the faces
// xi = +-1/2 are q0 + (a_k +- 3 b_k)/12 and at the Gauss points xi = s sqrt3/6 q0 + s (sqrt3/12) b_k
// (the two-point Gauss rule integrates the quadratic exactly, so its even part there is q0).
// The second differences are carried as sa_k = sqrt(13/3) a_k, which makes 4 beta_k two multiply-adds.
// P_k = prod_{j != k} (4 eps + 4 beta_j)^2: the nonlinear weights gamma_k / (eps + beta_k)^2,
// normalised, equal gamma_k P_k / sum_j gamma_j P_j (the common factor 4^4 cancels), so one reciprocal
// per evaluation point suffices.
// ---------------------------------------------------------------------------------------------
#define GKS_SA 2.0816659994661327  // sqrt(13/3)
template <typename real>
__device__ __forceinline__ void js_parts(real qm2, real qm1, real q0, real qp1, real qp2, real eps,
                                         real sa[3], real b[3], real P[3]) {
    const real d1 = qm1 - qm2, d2 = q0 - qm1, d3 = qp1 - q0, d4 = qp2 - qp1;
    const real s = real(GKS_SA), e4 = real(4) * eps;
    const real s2 = s * d2, s3 = s * d3;
    sa[0] = s2 - s * d1;
    b[0] = real(3) * d2 - d1;
    sa[1] = s3 - s2;
    b[1] = d2 + d3;
    sa[2] = s * d4 - s3;
    b[2] = real(3) * d3 - d4;
    real e[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        e[k] = fma_uniform(sa[k], sa[k], e4) + b[k] * b[k];
        e[k] *= e[k];
    }
    P[0] = e[1] * e[2];
    P[1] = e[0] * e[2];
    P[2] = e[0] * e[1];
}

// Face values of cell 0: right face (xi = +1/2, linear weights 1/10, 3/5, 3/10) and left face
// (xi = -1/2, weights 3/10, 3/5, 1/10). Both share the cell's smoothness indicators. The weights are
// divided by 3/5, and the 1/12 of the sub-stencil values and the scale of sa go into the denominator.
template <typename real>
__device__ __forceinline__ void weno_faces(real qm2, real qm1, real q0, real qp1, real qp2, real eps,
                                           real& right, real& left) {
    real sa[3], b[3], P[3];
    js_parts(qm2, qm1, q0, qp1, qp2, eps, sa, b, P);
    const real s3 = real(3 * GKS_SA);
    const real P1x = real(12 * GKS_SA) * P[1];
    real X0 = P[0] * (sa[0] + s3 * b[0]);
    real X1 = P[1] * (sa[1] + s3 * b[1]);
    real X2 = P[2] * (sa[2] + s3 * b[2]);
    right = q0 + (real(1.0 / 6.0) * X0 + (real(0.5) * X2 + X1)) *
                     rcp<real>(real(2 * GKS_SA) * P[0] + (real(6 * GKS_SA) * P[2] + P1x));
    X0 = P[0] * (sa[0] - s3 * b[0]);
    X1 = P[1] * (sa[1] - s3 * b[1]);
    X2 = P[2] * (sa[2] - s3 * b[2]);
    left = q0 + (real(0.5) * X0 + (real(1.0 / 6.0) * X2 + X1)) *
                    rcp<real>(real(6 * GKS_SA) * P[0] + (real(2 * GKS_SA) * P[2] + P1x));
}

// Linear weights at the Gauss points s = +-1 that reproduce the quartic: (7/36 - s sqrt3/1080, 11/18,
// 7/36 + s sqrt3/1080), here divided by 11/18 (WGL: the s = +1 outer weight of sub-stencil 0, WGH the
// other one).
#define GKS_WGL ((7.0 / 36.0 - GKS_SQRT3 / 1080.0) / (11.0 / 18.0))
#define GKS_WGH ((7.0 / 36.0 + GKS_SQRT3 / 1080.0) / (11.0 / 18.0))

// WENO-JS values at the two Gauss points of cell 0, vm (s = -1) and vp (s = +1). The sqrt3/12 of the
// sub-stencil deviations goes into the denominators.
template <typename real>
__device__ __forceinline__ void weno_gauss(real qm2, real qm1, real q0, real qp1, real qp2, real eps,
                                           real& vm, real& vp) {
    real a[3], b[3], P[3];
    js_parts(qm2, qm1, q0, qp1, qp2, eps, a, b, P);
    const real lo = real(GKS_WGL), hi = real(GKS_WGH), k = real(12.0 / GKS_SQRT3);
    const real X0 = P[0] * b[0], X1 = P[1] * b[1], X2 = P[2] * b[2];
    const real P1k = k * P[1];
    vp = q0 + (lo * X0 + (hi * X2 + X1)) * rcp<real>(real(k * lo) * P[0] + (real(k * hi) * P[2] + P1k));
    vm = q0 - (hi * X0 + (lo * X2 + X1)) * rcp<real>(real(k * hi) * P[0] + (real(k * lo) * P[2] + P1k));
}

// Quartic through five cell averages: values at the two Gauss points.
// value = e.q + s sqrt3 o.q, e = (-1/4320, 1/1080, 719/720, 1/1080, -1/4320),
// o = (7/432, -25/216, 0, 25/216, -7/432).
template <typename real>
__device__ __forceinline__ void quartic_gauss_value(real qm2, real qm1, real q0, real qp1, real qp2,
                                                    real& vm, real& vp) {
    real ev = real(-1.0 / 4320.0) * (qm2 + qp2) + real(1.0 / 1080.0) * (qm1 + qp1) + real(719.0 / 720.0) * q0;
    real od = real(GKS_SQRT3) * (real(7.0 / 432.0) * (qm2 - qp2) + real(25.0 / 216.0) * (qp1 - qm1));
    vm = ev - od;
    vp = ev + od;
}

// Quartic through five cell averages: derivatives (per unit cell) at the two Gauss points.
// e = (1/12, -2/3, 0, 2/3, -1/12), o = (-1/54, 13/54, -4/9, 13/54, -1/54).
template <typename real>
__device__ __forceinline__ void quartic_gauss_deriv(real qm2, real qm1, real q0, real qp1, real qp2,
                                                    real& dm, real& dp) {
    real ev = real(1.0 / 12.0) * (qm2 - qp2) + real(2.0 / 3.0) * (qp1 - qm1);
    real od = real(GKS_SQRT3) * (real(-1.0 / 54.0) * (qm2 + qp2) + real(13.0 / 54.0) * (qm1 + qp1) -
                                 real(4.0 / 9.0) * q0);
    dm = ev - od;
    dp = ev + od;
}

// The same with the coefficients scaled by the inverse width ih beforehand: three multiplications less, and on a
// uniform mesh the coefficients stay in scalar registers.
template <typename real>
struct QuarticDeriv {
    real e2, e1, o2, o1, o0;
    __device__ __forceinline__ explicit QuarticDeriv(real ih)
        : e2(real(1.0 / 12.0) * ih), e1(real(2.0 / 3.0) * ih), o2(real(-GKS_SQRT3 / 54.0) * ih),
          o1(real(GKS_SQRT3 * 13.0 / 54.0) * ih), o0(real(-GKS_SQRT3 * 4.0 / 9.0) * ih) {}
    __device__ __forceinline__ void operator()(real qm2, real qm1, real q0, real qp1, real qp2, real& dm, real& dp) const {
        const real ev = e2 * (qm2 - qp2) + e1 * (qp1 - qm1);
        const real od = o2 * (qm2 + qp2) + (o1 * (qm1 + qp1) + o0 * q0);
        dm = ev - od;
        dp = ev + od;
    }
};

// erf(a) - erf(b) without cancellation when a ~ b in FP32: three-point Gauss-Legendre quadrature of
// (2/sqrt(pi)) exp(-t^2) over [b, a] (relative error < 2e-8 for |a - b| < 1/4).
template <typename real>
__device__ __forceinline__ real erf_diff(real a, real b) {
    return Rc<real>::erf_(a) - Rc<real>::erf_(b);
}
template <>
__device__ __forceinline__ float erf_diff<float>(float a, float b) {
    float h = 0.5f * (a - b);
    if (fabsf(h) < 0.125f) {
        float m = 0.5f * (a + b);
        const float x1 = 0.77459666924148338f;  // sqrt(3/5)
        float t0 = m - h * x1, t2 = m + h * x1;
        float s = (5.0f / 9.0f) * (expf(-t0 * t0) + expf(-t2 * t2)) + (8.0f / 9.0f) * expf(-m * m);
        return 1.1283791670955126f * h * s;  // 2/sqrt(pi)
    }
    return erff(a) - erff(b);
}

// Maclaurin coefficients in y = x^2: erf x = (2/sqrt(pi)) x sum_k ERF[k] y^k, exp(-x^2) = sum_k EXP[k] y^k.
__device__ constexpr double KIN_ERF[10] = {1.0, -1.0 / 3.0, 0.1, -1.0 / 42.0, 1.0 / 216.0, -1.0 / 1320.0, 1.0 / 9360.0,
                                           -1.0 / 75600.0, 1.0 / 685440.0, -1.0 / 6894720.0};
__device__ constexpr double KIN_EXP[10] = {1.0, -1.0, 0.5, -1.0 / 6.0, 1.0 / 24.0, -1.0 / 120.0, 1.0 / 720.0,
                                           -1.0 / 5040.0, 1.0 / 40320.0, -1.0 / 362880.0};

// Polynomial P of degree N in A and its divided difference Q = (P(A) - P(B)) / (A - B): Horner's scheme at
// A leaves the coefficients of the quotient P(x) / (x - A), and Horner's scheme on those at B gives Q, so
// the pair costs 2 N - 1 multiply-adds and Q has no cancellation when A ~ B.
template <typename real, int N>
__device__ __forceinline__ void horner_pair(const double (&c)[10], real A, real B, real& PA, real& Q) {
    real r = real(c[N]), q;
    real rk[N];
#pragma unroll
    for (int k = N - 1; k >= 0; --k) {
        rk[k] = r;  // coefficient k of the quotient
        r = fma_uniform(A, r, real(c[k]));
    }
    PA = r;
    q = rk[N - 1];
#pragma unroll
    for (int k = N - 2; k >= 0; --k) q = fma(B, q, rk[k]);
    Q = q;
}

// Library form of kin_trans below. It is a call on purpose: flows inside the series' range never reach it,
// and its code inlined in the face kernels cost 60 registers and, in FP64, spills in their march (FP32: the tanh
// channel 1.3 % slower, the second-order variant 1.4 %).
template <typename real>
struct KinTrans {
    real hL, hR, hd, eR, dE;
};
template <typename real>
__device__ __attribute__((noinline)) KinTrans<real> kin_library(real aL, real aR) {
    KinTrans<real> k;
    k.hL = real(0.5) * (real(1) + Rc<real>::erf_(aL));
    k.hR = real(0.5) * (real(1) - Rc<real>::erf_(aR));
    k.hd = real(0.5) * erf_diff<real>(aL, aR);
    k.eR = Rc<real>::exp_(-aR * aR);
    k.dE = k.eR * Rc<real>::expm1_((aR - aL) * (aL + aR));
    return k;
}

// Transcendentals of the kinetic average at aL, aR: the half-space weights hL = (1 + erf aL) / 2 and
// hR = (1 - erf aR) / 2, half their excess hd = (erf aL - erf aR) / 2 = hL + hR - 1, the Gaussians
// eL = exp(-aL^2), eR = exp(-aR^2) and dE = eL - eR, the differences without cancellation.
// |aL|, |aR| <= 1/4 (|U_n| up to 0.35 of the sound speed, the flows of this scheme): with A = aL^2,
// B = aR^2 both functions are short polynomials in A and B,
//   erf aL - erf aR = (2/sqrt(pi)) (aL - aR) [P(A) + aR (aL + aR) Q],  P(B) = P(A) + (B - A) Q,
//   eL - eR = (A - B) Q_exp,  A - B = (aL - aR)(aL + aR).
// Truncation at |a| = 1/4, relative: FP32 (degrees 4 and 5) < 1e-9 in erf, 8e-9 in dE; FP64 (degree 9)
// < 1e-19 and 4e-17. Separate series of both arguments, a library exponential and expm1 took 36 FP32
// instructions more per Gauss point; the channel at 192 x 96 x 96 went from 0.922 to 0.902 ms a step in FP32
// and, with 12-term series and a library exponential gone, from 2.06 to 1.85 ms in FP64. Larger arguments
// take the library functions.
template <typename real>
__device__ __forceinline__ void kin_trans(real aL, real aR, real& hL, real& hR, real& hd, real& eL, real& eR,
                                          real& dE) {
    constexpr bool F32 = sizeof(real) == 4;
    const real dif = aL - aR, sum = aL + aR;
    if (__builtin_expect(fmax(fabs(aL), fabs(aR)) <= real(0.25), 1)) {
        constexpr int NP = F32 ? 4 : 9, NE = F32 ? 5 : 9;
        const real k1 = real(0.56418958354775628695);  // 1/sqrt(pi)
        const real A = aL * aL, B = aR * aR, AB = dif * sum;
        real PA, Q, QE;
        horner_pair<real, NP>(KIN_ERF, A, B, PA, Q);
        horner_pair<real, NE>(KIN_EXP, A, B, eL, QE);
        hL = fma(k1 * aL, PA, real(0.5));
        hR = fma(-k1 * aR, fma(-AB, Q, PA), real(0.5));
        hd = k1 * dif * fma(aR * sum, Q, PA);
        dE = AB * QE;
        eR = eL - dE;
    } else {
        const KinTrans<real> k = kin_library<real>(aL, aR);
        hL = k.hL;
        hR = k.hR;
        hd = k.hd;
        eR = k.eR;
        dE = k.dE;
        eL = eR + dE;
    }
}

template <typename real>
struct FluxConst {
    real lam;      // lambda = Ma^2 / (2 U_ref^2)
    real sl;       // sqrt(lambda)
    real kk;       // 1 / (2 sqrt(pi lambda))
    real c2;       // 1 / (2 lambda)
    real mu;       // viscosity
    real rho_ref;  // reference density
};

// Gas-kinetic flux at one Gauss point, in the face's local frame: variables (rho', m_n, m_t1, m_t2),
// derivative directions (n, t1, t2). qL, qR: reconstructed left/right states; g[d][v]: dQ_v/dx_d.
// Gives F0 (if NEED_F0) and F1 (the caller sums them and applies the quadrature weight).
// SHIFT: qL[1], qR[1] hold m_n - cm for a constant cm, and the mass-flux part of f0 receives F0 - cm
// (the constant cancels in the flux difference of a cell). The half-space weights satisfy
// hL + hR - 1 = (erf(aL) - erf(aR)) / 2, so the shifted mass flux carries no O(cm) rounding.
template <typename real, bool NEED_F0, bool SHIFT = false>
__device__ __forceinline__ void gp_flux(const real qL[4], const real qR[4], const real g[3][4],
                                        const FluxConst<real>& k, real f0[4], real f1[4], real cm = real(0)) {
    // kinetic (half-space) average of the left and right Maxwellians, in deviation form
    const real rL = k.rho_ref + qL[0], rR = k.rho_ref + qR[0];
    const real mL = SHIFT ? cm + qL[1] : qL[1], mR = SHIFT ? cm + qR[1] : qR[1];
    const real aL = k.sl * (mL * rcp<real>(rL)), aR = k.sl * (mR * rcp<real>(rR));
    real hL, hR, hd, eL, eR, dE;
    kin_trans<real>(aL, aR, hL, hR, hd, eL, eR, dE);
    const real rho0p = qL[0] * hL + (qR[0] * hR + k.rho_ref * hd);
    // F0 of the density: m0[0], or m0[0] - cm when shifted
    real mass_flux = qL[1] * hL + (qR[1] * hR + k.kk * (qL[0] * eL - (qR[0] * eR - k.rho_ref * dE)));
    if (SHIFT) mass_flux += cm * hd;
    real m0[3];
    m0[0] = SHIFT ? cm + mass_flux : mass_flux;
    m0[1] = qL[2] * hL + qR[2] * hR;
    m0[2] = qL[3] * hL + qR[3] * hR;
    const real ir = rcp<real>(k.rho_ref + rho0p);
    const real U[3] = {m0[0] * ir, m0[1] * ir, m0[2] * ir};
    if (NEED_F0) {
        // the velocity gradients of the stress, times rho0: r_dj = dm_j/dx_d - U_j drho/dx_d
        const real mi = k.mu * ir;
        const real s00 = real(2) * (g[0][1] - U[0] * g[0][0]);
        const real s01 = (g[0][2] + g[1][1]) - U[1] * g[0][0] - U[0] * g[1][0];
        const real s02 = (g[0][3] + g[2][1]) - U[2] * g[0][0] - U[0] * g[2][0];
        f0[0] = mass_flux;
        f0[1] = (m0[0] * U[0] + k.c2 * rho0p) - mi * s00;
        f0[2] = m0[0] * U[1] - mi * s01;
        f0[3] = m0[0] * U[2] - mi * s02;
    }
    // Euler time derivative of Q0. Its advection term needs no velocity gradient:
    // rho0 (U . grad) U_j = sum_d U_d dm_j/dx_d - U_j sum_d U_d drho/dx_d.
    const real qd0 = -((g[0][1] + g[1][2]) + g[2][3]);
    const real H = U[0] * g[0][0] + (U[1] * g[1][0] + (U[2] * g[2][0] + qd0));
    real qd[3];
#pragma unroll
    for (int j = 0; j < 3; ++j)
        qd[j] = U[j] * H - (U[0] * g[0][1 + j] + (U[1] * g[1][1 + j] + (U[2] * g[2][1 + j] + k.c2 * g[j][0])));
    const real tn = qd[0] - U[0] * qd0;  // rho0 dU_n/dt
    f1[0] = qd[0];
    f1[1] = U[0] * (qd[0] + tn) + k.c2 * qd0;
    f1[2] = U[1] * tn + U[0] * qd[1];
    f1[3] = U[2] * tn + U[0] * qd[2];
}

// ---------------------------------------------------------------------------------------------
// Adjoint support (FP64): WENO evaluations that also return their normalised nonlinear weights, the
// sub-stencil coefficients those weights combine, and the reverse of gp_flux.
// ---------------------------------------------------------------------------------------------
template <typename real>
__device__ __forceinline__ void weno_faces_w(real qm2, real qm1, real q0, real qp1, real qp2, real eps,
                                             real& right, real& left, real wr[3], real wl[3]) {
    real a[3], b[3], P[3];  // a: scaled by GKS_SA
    js_parts(qm2, qm1, q0, qp1, qp2, eps, a, b, P);
    const real s3 = real(3 * GKS_SA), ia = real(1.0 / GKS_SA);
    // weights divided by 3/5 and multiplied by 12 in the denominator, as in weno_faces
    const real P1x = real(12) * P[1];
    real c0 = real(2) * P[0], c2 = real(6) * P[2];
    real is = rcp<real>(c0 + (c2 + P1x));
    wr[0] = c0 * is;
    wr[1] = P1x * is;
    wr[2] = c2 * is;
    right = q0 + (real(1.0 / 6.0) * P[0] * (a[0] + s3 * b[0]) +
                  (real(0.5) * P[2] * (a[2] + s3 * b[2]) + P[1] * (a[1] + s3 * b[1]))) * (ia * is);
    c0 = real(6) * P[0];
    c2 = real(2) * P[2];
    is = rcp<real>(c0 + (c2 + P1x));
    wl[0] = c0 * is;
    wl[1] = P1x * is;
    wl[2] = c2 * is;
    left = q0 + (real(0.5) * P[0] * (a[0] - s3 * b[0]) +
                 (real(1.0 / 6.0) * P[2] * (a[2] - s3 * b[2]) + P[1] * (a[1] - s3 * b[1]))) * (ia * is);
}

template <typename real>
__device__ __forceinline__ void weno_gauss_w(real qm2, real qm1, real q0, real qp1, real qp2, real eps,
                                             real& vm, real& vp, real wm[3], real wp[3]) {
    real a[3], b[3], P[3];
    js_parts(qm2, qm1, q0, qp1, qp2, eps, a, b, P);
    const real lo = real(GKS_WGL), hi = real(GKS_WGH), r12 = real(GKS_SQRT3 / 12.0);
    const real X0 = P[0] * b[0], X1 = P[1] * b[1], X2 = P[2] * b[2];
    real c0 = lo * P[0], c2 = hi * P[2];
    real is = rcp<real>(c0 + (c2 + P[1]));
    wp[0] = c0 * is;
    wp[1] = P[1] * is;
    wp[2] = c2 * is;
    vp = q0 + r12 * (lo * X0 + (hi * X2 + X1)) * is;
    c0 = hi * P[0];
    c2 = lo * P[2];
    is = rcp<real>(c0 + (c2 + P[1]));
    wm[0] = c0 * is;
    wm[1] = P[1] * is;
    wm[2] = c2 * is;
    vm = q0 - r12 * (hi * X0 + (lo * X2 + X1)) * is;
}

// Coefficient of cell r (0..4 over the stencil -2..2) in sub-stencil k's value:
//   face xi = +1/2 (side 0) and xi = -1/2 (side 1); Gauss point s = -1 (side 2) and s = +1 (side 3).
__device__ __forceinline__ double sub_coef(int side, int k, int r) {
    const int l = r - k;
    if (l < 0 || l > 2) return 0.0;
    const double t = GKS_SQRT3;
    switch (side) {
        case 0: {
            const double c[3][3] = {{2.0 / 6, -7.0 / 6, 11.0 / 6}, {-1.0 / 6, 5.0 / 6, 2.0 / 6}, {2.0 / 6, 5.0 / 6, -1.0 / 6}};
            return c[k][l];
        }
        case 1: {
            const double c[3][3] = {{-1.0 / 6, 5.0 / 6, 2.0 / 6}, {2.0 / 6, 5.0 / 6, -1.0 / 6}, {11.0 / 6, -7.0 / 6, 2.0 / 6}};
            return c[k][l];
        }
        default: {
            const double s = side == 2 ? -1.0 : 1.0;
            const double c[3][3] = {{s * t / 12, -s * t / 3, 1.0 + s * t / 4},
                                    {-s * t / 12, 1.0, s * t / 12},
                                    {1.0 - s * t / 4, s * t / 3, -s * t / 12}};
            return c[k][l];
        }
    }
}

// Effective linear weight of stencil cell r for nonlinear weights w[3] on a given side.
__device__ __forceinline__ double weno_eff(int side, const double w[3], int r) {
    return w[0] * sub_coef(side, 0, r) + w[1] * sub_coef(side, 1, r) + w[2] * sub_coef(side, 2, r);
}

// Jacobian row dv/dq_r (r = 0..4 over the stencil -2..2) of a WENO-JS evaluation on `side` (as in
// sub_coef) with the nonlinear weights differentiated too. With e_k = 4 (eps + beta_k) the normalised
// weights are omega_k = (gamma_k / e_k^2) / sum_j (gamma_j / e_j^2), so
//   dv/dq_r = sum_k omega_k c_k[r] - 2 sum_k omega_k (v_k - v) (de_k/dq_r) / e_k,
// v_k the sub-stencil values and c_k[r] their coefficients. w: the weights, v: the value.
__device__ __forceinline__ void weno_jacobian(int side, const double q[5], double eps, const double w[3], double v,
                                              double J[5]) {
    const double c133 = 13.0 / 3.0, e4 = 4.0 * eps;
    // 4 beta_k = (13/3) a_k^2 + b_k^2 with a_k, b_k linear in the sub-stencil's cells
    const double a0 = q[0] - 2.0 * q[1] + q[2], b0 = q[0] - 4.0 * q[1] + 3.0 * q[2];
    const double a1 = q[1] - 2.0 * q[2] + q[3], b1 = q[1] - q[3];
    const double a2 = q[2] - 2.0 * q[3] + q[4], b2 = 3.0 * q[2] - 4.0 * q[3] + q[4];
    const double e[3] = {e4 + c133 * a0 * a0 + b0 * b0, e4 + c133 * a1 * a1 + b1 * b1, e4 + c133 * a2 * a2 + b2 * b2};
    double g[3];
    for (int k = 0; k < 3; ++k) {
        double vk = 0.0;
        for (int l = 0; l < 3; ++l) vk += sub_coef(side, k, k + l) * q[k + l];
        g[k] = -2.0 * w[k] * (vk - v) / e[k];
    }
    // de_k/dq over the sub-stencil's three cells: (26/3) a (1, -2, 1) + 2 b (db/dq)
    const double t0 = 26.0 / 3.0 * a0, t1 = 26.0 / 3.0 * a1, t2 = 26.0 / 3.0 * a2;
    const double d0[3] = {t0 + 2.0 * b0, -2.0 * t0 - 8.0 * b0, t0 + 6.0 * b0};
    const double d1[3] = {t1 + 2.0 * b1, -2.0 * t1, t1 - 2.0 * b1};
    const double d2[3] = {t2 + 6.0 * b2, -2.0 * t2 - 8.0 * b2, t2 + 2.0 * b2};
    for (int r = 0; r < 5; ++r) J[r] = weno_eff(side, w, r);
    for (int l = 0; l < 3; ++l) {
        J[l] += g[0] * d0[l];
        J[1 + l] += g[1] * d1[l];
        J[2 + l] += g[2] * d2[l];
    }
}

// Quartic Gauss value (deriv = 0) or derivative (deriv = 1) coefficient of stencil cell r at s.
__device__ __forceinline__ double quartic_coef(int deriv, int s, int r) {
    const double t = GKS_SQRT3;
    if (deriv == 0) {
        const double e[5] = {-1.0 / 4320, 1.0 / 1080, 719.0 / 720, 1.0 / 1080, -1.0 / 4320};
        const double o[5] = {7.0 / 432, -25.0 / 216, 0.0, 25.0 / 216, -7.0 / 432};
        return e[r] + s * t * o[r];
    }
    const double e[5] = {1.0 / 12, -2.0 / 3, 0.0, 2.0 / 3, -1.0 / 12};
    const double o[5] = {-1.0 / 54, 13.0 / 54, -4.0 / 9, 13.0 / 54, -1.0 / 54};
    return e[r] + s * t * o[r];
}

// Reverse of gp_flux (FP64): given the adjoints b0 (of the accumulated F0 contribution, stage 1
// only) and b1 (of F1), add the adjoints of the Gauss-point inputs to qLb, qRb, gb.
template <bool NEED_F0>
__device__ __forceinline__ void gp_flux_adj(const double qL[4], const double qR[4], const double g[3][4],
                                            const FluxConst<double>& k, double w, const double b0[4],
                                            const double b1[4], double qLb[4], double qRb[4], double gb[3][4]) {
    // ---- forward recompute
    const double rL = k.rho_ref + qL[0], rR = k.rho_ref + qR[0];
    const double irL = rcp<double>(rL), irR = rcp<double>(rR);
    const double uL = qL[1] * irL, uR = qR[1] * irR;
    const double aL = k.sl * uL, aR = k.sl * uR;
    // the forward's evaluation of the half-space weights and Gaussians
    double hL, hR, hd, eL, eR, dE;
    kin_trans<double>(aL, aR, hL, hR, hd, eL, eR, dE);
    const double rho0p = qL[0] * hL + qR[0] * hR + k.rho_ref * hd;
    double m0[3];
    m0[0] = qL[1] * hL + qR[1] * hR + k.kk * (qL[0] * eL - qR[0] * eR + k.rho_ref * dE);
    m0[1] = qL[2] * hL + qR[2] * hR;
    m0[2] = qL[3] * hL + qR[3] * hR;
    const double r0 = k.rho_ref + rho0p;
    const double ir = rcp<double>(r0);
    double U[3] = {m0[0] * ir, m0[1] * ir, m0[2] * ir};
    double dU[3][3];
    for (int d = 0; d < 3; ++d)
        for (int j = 0; j < 3; ++j) dU[d][j] = (g[d][1 + j] - U[j] * g[d][0]) * ir;
    const double divm = g[0][1] + g[1][2] + g[2][3];
    const double qd0 = -divm;
    double adv[3], qd[3];
    for (int j = 0; j < 3; ++j) {
        adv[j] = U[0] * dU[0][j] + U[1] * dU[1][j] + U[2] * dU[2][j];
        qd[j] = -U[j] * divm - r0 * adv[j] - k.c2 * g[j][0];
    }
    // ---- reverse
    double A1[4], A0[4];
    for (int v = 0; v < 4; ++v) {
        A1[v] = w * b1[v];
        A0[v] = NEED_F0 ? w * b0[v] : 0.0;
    }
    double Ub[3] = {0, 0, 0}, m0b[3] = {0, 0, 0}, dUb[3][3] = {{0, 0, 0}, {0, 0, 0}, {0, 0, 0}};
    double qdb[3] = {0, 0, 0};
    double qd0b = 0.0, r0b = 0.0, r0pb = 0.0, irb = 0.0, divmb = 0.0;
    // F1
    qdb[0] += A1[0];
    Ub[0] += A1[1] * (2.0 * qd[0] - 2.0 * U[0] * qd0);
    qdb[0] += A1[1] * 2.0 * U[0];
    qd0b += A1[1] * (-U[0] * U[0] + k.c2);
    for (int j = 1; j < 3; ++j) {
        Ub[j] += A1[1 + j] * (qd[0] - U[0] * qd0);
        Ub[0] += A1[1 + j] * (qd[j] - U[j] * qd0);
        qdb[0] += A1[1 + j] * U[j];
        qdb[j] += A1[1 + j] * U[0];
        qd0b += -A1[1 + j] * U[0] * U[j];
    }
    double advb[3];
    for (int j = 0; j < 3; ++j) {
        Ub[j] += -qdb[j] * divm;
        divmb += -qdb[j] * U[j];
        r0b += -qdb[j] * adv[j];
        advb[j] = -qdb[j] * r0;
        gb[j][0] += -k.c2 * qdb[j];
    }
    for (int j = 0; j < 3; ++j)
        for (int d = 0; d < 3; ++d) {
            Ub[d] += advb[j] * dU[d][j];
            dUb[d][j] += advb[j] * U[d];
        }
    divmb += -qd0b;
    gb[0][1] += divmb;
    gb[1][2] += divmb;
    gb[2][3] += divmb;
    // F0
    if (NEED_F0) {
        m0b[0] += A0[0];
        m0b[0] += A0[1] * U[0];
        Ub[0] += A0[1] * m0[0];
        r0pb += A0[1] * k.c2;
        dUb[0][0] += -2.0 * k.mu * A0[1];
        for (int j = 1; j < 3; ++j) {
            m0b[0] += A0[1 + j] * U[j];
            Ub[j] += A0[1 + j] * m0[0];
            dUb[0][j] += -k.mu * A0[1 + j];
            dUb[j][0] += -k.mu * A0[1 + j];
        }
    }
    // velocity gradients
    for (int d = 0; d < 3; ++d)
        for (int j = 0; j < 3; ++j) {
            gb[d][1 + j] += dUb[d][j] * ir;
            Ub[j] += -dUb[d][j] * g[d][0] * ir;
            gb[d][0] += -dUb[d][j] * U[j] * ir;
            irb += dUb[d][j] * dU[d][j] * r0;
        }
    for (int j = 0; j < 3; ++j) {
        m0b[j] += Ub[j] * ir;
        irb += Ub[j] * m0[j];
    }
    r0b += -irb * ir * ir;
    r0pb += r0b;
    // kinetic average
    double hLb = 0.0, hRb = 0.0, eLb = 0.0, eRb = 0.0, EaLb = 0.0, EaRb = 0.0;
    for (int j = 1; j < 3; ++j) {
        qLb[1 + j] += m0b[j] * hL;
        qRb[1 + j] += m0b[j] * hR;
        hLb += m0b[j] * qL[1 + j];
        hRb += m0b[j] * qR[1 + j];
    }
    qLb[1] += m0b[0] * hL;
    qRb[1] += m0b[0] * hR;
    hLb += m0b[0] * qL[1];
    hRb += m0b[0] * qR[1];
    qLb[0] += m0b[0] * k.kk * eL;
    qRb[0] += -m0b[0] * k.kk * eR;
    eLb += m0b[0] * k.kk * (qL[0] + k.rho_ref);
    eRb += -m0b[0] * k.kk * (qR[0] + k.rho_ref);
    qLb[0] += r0pb * hL;
    qRb[0] += r0pb * hR;
    hLb += r0pb * qL[0];
    hRb += r0pb * qR[0];
    EaLb += 0.5 * k.rho_ref * r0pb;
    EaRb += -0.5 * k.rho_ref * r0pb;
    EaLb += 0.5 * hLb;
    EaRb += -0.5 * hRb;
    const double c2pi = 1.1283791670955126;  // 2 / sqrt(pi)
    // d erf(sl u)/du = sl (2/sqrt(pi)) exp(-sl^2 u^2), and sl^2 = lambda: exp(-aL^2) is eL
    double uLb = k.sl * EaLb * c2pi * eL + eLb * eL * (-2.0 * k.lam * uL);
    double uRb = k.sl * EaRb * c2pi * eR + eRb * eR * (-2.0 * k.lam * uR);
    qLb[1] += uLb * irL;
    qLb[0] += -uLb * qL[1] * irL * irL;
    qRb[1] += uRb * irR;
    qRb[0] += -uRb * qR[1] * irR * irR;
}

}  // namespace gks
