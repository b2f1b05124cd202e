// Device-side building blocks of the finite-volume step for gfx950:
// geometry of the ghosted SoA layout, integer division by an invariant,
// the minmod MUSCL face states and the Roe flux.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace fvk {

constexpr int NG = 2;  // ghost layers per face (the 4-cell MUSCL stencil)

// Division by a run-time invariant d >= 1 for 0 <= n < 2^32, by multiply-high
// and shifts (Granlund & Montgomery, "Division by invariant integers using
// multiplication", PLDI 1994, unsigned case).
struct DivMod {
    uint32_t d, m, sh1, sh2;
};

inline DivMod make_divmod(uint32_t d) {
    uint32_t l = 0;
    while ((1ull << l) < d) ++l;  // l = ceil(log2 d)
    DivMod r;
    r.d = d;
    r.m = (uint32_t)((((1ull << l) - d) << 32) / d + 1);
    r.sh1 = l < 1 ? l : 1;
    r.sh2 = l > 0 ? l - 1 : 0;
    return r;
}

__host__ __device__ inline uint32_t divq(uint32_t n, const DivMod& dm) {
    uint32_t t = (uint32_t)(((uint64_t)dm.m * n) >> 32);
    return (t + ((n - t) >> dm.sh1)) >> dm.sh2;
}

// Geometry and constants of one grid, passed by value to every kernel.
// Ghost state of inflow faces, per axis and side (conserved variables).
struct BcState {
    double q[3][2][5];
};

struct Geo {
    int ndim, nvar;
    int n[3];           // interior cells per axis
    int sy, sz;         // state strides in elements (s_x = 1)
    int off0;           // offset of interior cell (0,0,0) inside one variable
    int ncell;          // n[0] * n[1] * n[2]
    long long sv;       // per-variable stride of the state
    long long fsv[3];   // per-variable stride of the face-flux array of each axis
    DivMod dnx, dny;    // division by n[0] and n[1]
    double inv_dx[3];   // 1 / dx_d
    double area[3];     // face area of axis d: product of the other widths
    double inv_vol;     // 1 / |Omega|
    double vol;         // |Omega|
    double gamma, gm1;  // gamma, gamma - 1
    double cfl;
    int bc[3][2];
    int scheme;         // 0 minmod; Psi = 1 with kappa = -1, 0, 1/3, 1 for 1 .. 4; 5 van Leer; 6 kappa = 1/2
    double mu;          // dynamic viscosity, 0 for the Euler equations
    double kcond;       // heat conductivity mu gamma / ((gamma - 1) Pr)
    double nu_fac;      // max(4/3, gamma / Pr): the larger diffusivity per unit kinematic viscosity
    // Curvilinear 2D grid (null for the uniform box): metric streams in the
    // workspace, SoA. x faces ((nx + 1) ny each, face (i, j) between cells
    // (i - 1, j) and (i, j)): unit normal x, unit normal y, length; then y
    // faces (nx (ny + 1) each, face (i, j) between (i, j - 1) and (i, j)): the
    // same three; then per cell: area and 1 / area.
    const double* met;
};

// Offsets of the metric streams of a curvilinear grid (elements).
struct MetricOffsets {
    long long fx, fy, cell;  // first element of the x-face, y-face and cell blocks
    long long nfx, nfy, nc;  // entries per stream of each block
};

__host__ __device__ inline MetricOffsets metric_offsets(int nx, int ny) {
    MetricOffsets m;
    m.nfx = (long long)(nx + 1) * ny;
    m.nfy = (long long)nx * (ny + 1);
    m.nc = (long long)nx * ny;
    m.fx = 0;
    m.fy = 3 * m.nfx;
    m.cell = m.fy + 3 * m.nfy;
    return m;
}

// 1/a and 1/sqrt(a) for the flux arithmetic: the hardware estimates
// (v_rcp_f64, v_rsq_f64, relative error about 5e-8) refined by one
// third-order correction each. With e the residual of the estimate y0,
//   1/a       = y0 / (1 - e)      = y0 (1 + e + e^2 + ...),        e = 1 - a y0,
//   1/sqrt(a) = y0 (1 - e)^(-1/2) = y0 (1 + e/2 + 3e^2/8 + ...),  e = 1 - a y0^2,
// and the series is cut after e^2, leaving an error of order e^3 (below
// 1e-21) plus the rounding of the last fma: within about one ulp of the
// correctly rounded result for the normal, positive arguments the Euler
// fluxes produce, in 3 (rcp) and 5 (rsqrt) operations after the estimate.
__host__ __device__ __forceinline__ double rcp_nr(double a) {
#if defined(__HIP_DEVICE_COMPILE__)
    const double x = __builtin_amdgcn_rcp(a);
    const double e = fma(-a, x, 1.0);
    return fma(x, fma(e, e, e), x);
#else
    return 1.0 / a;
#endif
}

__host__ __device__ __forceinline__ double rsqrt_nr(double a) {
#if defined(__HIP_DEVICE_COMPILE__)
    const double y = __builtin_amdgcn_rsq(a);
    const double e = fma(-a * y, y, 1.0);
    return fma(y * e, fma(0.375, e, 0.5), y);
#else
    return 1.0 / sqrt(a);
#endif
}

// minmod(a, b): zero unless a and b share a strict sign, else the one of smaller
// magnitude, i.e. the median of a, b and 0, written as
// max(min(a, b), min(max(a, b), 0)): for two positive slopes the inner min
// with 0 gives 0 and the outer max the smaller slope, for two negative ones
// the inner min gives the one nearer 0, and for mixed signs or a zero the
// result is 0. No product, so tiny slopes do not underflow, and no compares
// or selects (four min/max).
__host__ __device__ __forceinline__ double minmod(double a, double b) {
    return fmax(fmin(a, b), fmin(fmax(a, b), 0.0));
}

// van Leer's limited difference Psi(b/a) a with Psi(r) = (r + |r|)/(1 + |r|):
// 2ab/(a + b) for slopes of one sign, else 0. Symmetric in a and b, bit for
// bit (products and sums commute), so one value serves both faces of a cell.
__host__ __device__ __forceinline__ double vanleer(double a, double b) {
    const double ab = a * b;
    return ab > 0.0 ? 2.0 * ab * rcp_nr(a + b) : 0.0;
}

// MUSCL face states from the three differences of the stencil,
// dm = q1 - q0, dc = q2 - q1, dp = q3 - q2 (for callers that share them
// between neighbouring faces); UNL selects Psi = 1.
template <bool UNL>
__host__ __device__ __forceinline__ void muscl_from_diffs(double q1, double q2, double dm, double dc, double dp,
                                                         double& qL, double& qR) {
    if (UNL) {
        qL = q1 + 0.5 * dm;
        qR = q2 - 0.5 * dp;
    } else {
        qL = q1 + 0.5 * minmod(dm, dc);
        qR = q2 - 0.5 * minmod(dp, dc);
    }
}

// MUSCL face states (epsilon = 1, kappa = -1, minmod) at face k+1/2 of the
// cells q0 = k-1, q1 = k, q2 = k+1, q3 = k+2.
__host__ __device__ __forceinline__ void muscl_minmod(double q0, double q1, double q2, double q3,
                                             double& qL, double& qR) {
    muscl_from_diffs<false>(q1, q2, q1 - q0, q2 - q1, q3 - q2, qL, qR);
}

// The same with the choice fixed at compile time (UNL: Psi = 1), for loops
// that must stay free of branches.
template <bool UNL>
__host__ __device__ __forceinline__ void muscl_fixed(double q0, double q1, double q2, double q3, double& qL,
                                                    double& qR) {
    muscl_from_diffs<UNL>(q1, q2, q1 - q0, q2 - q1, q3 - q2, qL, qR);
}

// Weights of the unlimited (Psi = 1) kappa family of Eq. (flux) with
// epsilon = 1: Q^L = Q_k + a dQ_{k-1/2} + b dQ_{k+1/2} and
// Q^R = Q_{k+1} - b dQ_{k+1/2} - a dQ_{k+3/2}, a = (1 - kappa)/4,
// b = (1 + kappa)/4, for schemes 2 .. 4 (kappa = 0, 1/3, 1) and 6 (kappa = 1/2).
__host__ __device__ __forceinline__ void kappa_weights(int scheme, double& a, double& b) {
    const double kappa = scheme == 2 ? 0.0 : (scheme == 3 ? 1.0 / 3.0 : (scheme == 6 ? 0.5 : 1.0));
    a = 0.25 * (1.0 - kappa);
    b = 0.25 * (1.0 + kappa);
}

// Face states of the kappa family from the stencil's differences, with
// explicit fused multiply-adds: the same bits whether the differences are
// formed per face or shared per cell, whatever the compiler contracts.
__host__ __device__ __forceinline__ void muscl_kappa_diffs(double q1, double q2, double dm, double dc, double dp,
                                                          double a, double b, double& qL, double& qR) {
    qL = fma(a, dm, fma(b, dc, q1));
    qR = fma(-b, dc, fma(-a, dp, q2));
}

// The same with the scheme chosen at run time (uniform): 0 minmod, 1 Psi = 1
// with kappa = -1, 2 .. 4 and 6 the other kappa members, 5 van Leer.
__host__ __device__ __forceinline__ void muscl(double q0, double q1, double q2, double q3, int scheme,
                                              double& qL, double& qR) {
    if (scheme == 1) {
        qL = q1 + 0.5 * (q1 - q0);
        qR = q2 - 0.5 * (q3 - q2);
    } else if (scheme == 0) {
        muscl_minmod(q0, q1, q2, q3, qL, qR);
    } else if (scheme == 5) {
        const double dc = q2 - q1;
        qL = q1 + 0.5 * vanleer(q1 - q0, dc);
        qR = q2 - 0.5 * vanleer(dc, q3 - q2);
    } else {
        double a, b;
        kappa_weights(scheme, a, b);
        muscl_kappa_diffs(q1, q2, q1 - q0, q2 - q1, q3 - q2, a, b, qL, qR);
    }
}

// x with its sign bit set where r's is: a negative density makes the product
// of the two densities negative whatever the other's sign, so that its root
// is NaN and the flux carries it.
__host__ __device__ __forceinline__ double sign_from(double x, double r) {
#if defined(__HIP_DEVICE_COMPILE__)
    const long long b = __double_as_longlong(x), n = __double_as_longlong(r);
    const uint32_t hi = (uint32_t)(b >> 32) | ((uint32_t)(n >> 32) & 0x80000000u);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | (uint32_t)b));
#else
    return r < 0.0 ? -fabs(x) : x;
#endif
}

// Roe flux along axis AX for NDIM dimensions, conserved face states in, flux out.
// F = (F(qL) + F(qR))/2 - sum_k |lambda_k| alpha_k r_k / 2, no entropy fix.
// TWICE returns 2F: callers that difference the fluxes fold the exact factor
// 1/2 into their face areas and save a multiply per component.
//
// The vector ALU bounds every kernel that evaluates it, so the operations are
// counted: 86 in 2D, 3 of them reciprocal estimates at a quarter of the rate
// (102 with 4 estimates when written by wave strengths).
//  - One root serves both densities: with y = (rL rR)^(-1/2), 1/rL = rR y^2,
//    1/rR = rL y^2, the averaged density is rL rR y, and the Roe weight of the
//    right state is sqrt(rR) / (sqrt(rL) + sqrt(rR)) = rR / (rR + rho~). The
//    product of the densities and its inverse have to be normal numbers: their
//    geometric mean lies between 1e-153 and 1e153 (a root for each density took
//    any normal one).
//  - The dissipation is |u_n| dU plus an acoustic part. With m = min(|u_n| / c, 1)
//    (the two acoustic speeds' half sum is max(|u_n|, c), their half difference
//    u_n clamped to +-c), s = m with u_n's sign and t = c (1 - m):
//      A = (t / c^2) dp + s rho~ du_n,  B = s dp + t rho~ du_n  (t / c^2 = (1 - m) / c),
//      D = |u_n| dU + A (1, u~, H~) + B (0, n, u~_n).
// Fused multiply-adds are written out and nothing else is contracted: the same
// bits in every kernel that evaluates a face.
template <int NDIM, int AX, bool TWICE = false>
__host__ __device__ __forceinline__ void roe_flux(const double* qL, const double* qR, double gm1, double* F) {
#pragma clang fp contract(off)
    constexpr int IE = NDIM + 1;
    const double rL = qL[0], rR = qR[0];
    const double rr = sign_from(rL * rR, rL);
    const double y = rsqrt_nr(rr);
    const double y2 = y * y;
    const double irL = rR * y2, irR = rL * y2;
    const double rt = rr * y;
    const double wR = rR * rcp_nr(rR + rt);
    // velocities, pressures, total enthalpies
    double uL[NDIM], uR[NDIM];
#pragma unroll
    for (int d = 0; d < NDIM; ++d) {
        uL[d] = qL[1 + d] * irL;
        uR[d] = qR[1 + d] * irR;
    }
    double keL = qL[1] * uL[0], keR = qR[1] * uR[0];
#pragma unroll
    for (int d = 1; d < NDIM; ++d) {
        keL = fma(qL[1 + d], uL[d], keL);
        keR = fma(qR[1 + d], uR[d], keR);
    }
    const double pL = gm1 * fma(-0.5, keL, qL[IE]);
    const double pR = gm1 * fma(-0.5, keR, qR[IE]);
    const double hL = qL[IE] + pL, hR = qR[IE] + pR;
    const double HL = hL * irL, HR = hR * irR;
    // Roe averages
    double ut[NDIM];
#pragma unroll
    for (int d = 0; d < NDIM; ++d) ut[d] = fma(wR, uR[d] - uL[d], uL[d]);
    double qqt = ut[0] * ut[0];
#pragma unroll
    for (int d = 1; d < NDIM; ++d) qqt = fma(ut[d], ut[d], qqt);
    const double Ht = fma(wR, HR - HL, HL);
    const double c2 = gm1 * fma(-0.5, qqt, Ht);
    const double rc = rsqrt_nr(c2);
    const double c = c2 * rc;
    const double un = ut[AX], aun = fabs(un);
    // acoustic part
    const double m = fmin(fmax(aun * rc, 0.0), 1.0);
    const double sm = copysign(m, un);
    const double dp = pR - pL;
    const double rdu = rt * (uR[AX] - uL[AX]);
    const double A = fma(fma(-rc, m, rc), dp, sm * rdu);
    const double B = fma(sm, dp, fma(-c, m, c) * rdu);
    // fluxes of both sides (the mass flux rho u_n is the normal momentum itself) minus the dissipation
    const double mL = qL[1 + AX], mR = qR[1 + AX];
    constexpr double h = TWICE ? 1.0 : 0.5;
    F[0] = h * (fma(-aun, rR - rL, mL + mR) - A);
#pragma unroll
    for (int d = 0; d < NDIM; ++d) {
        double f = d == AX ? fma(mR, uR[d], fma(mL, uL[d], pL + pR)) : fma(mR, uR[d], mL * uL[d]);
        f = fma(-A, ut[d], fma(-aun, qR[1 + d] - qL[1 + d], f));
        F[1 + d] = h * (d == AX ? f - B : f);
    }
    F[IE] = h * fma(-B, un, fma(-A, Ht, fma(-aun, qR[IE] - qL[IE], fma(hR, uR[AX], hL * uL[AX]))));
}

// Roe flux through a 2D face of unit normal (nx, ny), conserved face states
// in, flux out: the momenta are turned into the face's frame (normal
// nx u + ny v, tangential -ny u + nx v), the flux of the x-axis form above is
// taken there, and its momentum part is turned back. The same flux as the
// normal form F = (F_n(QL) + F_n(QR))/2 - |A_n| dQ / 2 with V_n = n.u.
__host__ __device__ __forceinline__ void roe_flux_n2(const double* qL, const double* qR, double nx, double ny,
                                                     double gm1, double* F) {
    double a[4], b[4], G[4];
    a[0] = qL[0];
    a[1] = nx * qL[1] + ny * qL[2];
    a[2] = -ny * qL[1] + nx * qL[2];
    a[3] = qL[3];
    b[0] = qR[0];
    b[1] = nx * qR[1] + ny * qR[2];
    b[2] = -ny * qR[1] + nx * qR[2];
    b[3] = qR[3];
    roe_flux<2, 0>(a, b, gm1, G);
    F[0] = G[0];
    F[1] = nx * G[1] - ny * G[2];
    F[2] = ny * G[1] + nx * G[2];
    F[3] = G[3];
}

// Wave-speed bound of one cell, sum_d (|u_d| + c) * inv_dx[d], and the
// non-physical flags (1 NaN, 2 rho <= 0, 4 p <= 0) it raises.
template <int NDIM>
__host__ __device__ __forceinline__ double cell_lambda(const double* q, double gamma, double gm1, const double* inv_dx,
                                                       uint32_t& fl) {
    constexpr int IE = NDIM + 1;
    const double rho = q[0];
    const double ir = rcp_nr(rho);
    double u[NDIM];
    double qq = 0.0;
    for (int d = 0; d < NDIM; ++d) {
        u[d] = q[1 + d] * ir;
        qq += u[d] * u[d];
    }
    const double p = gm1 * (q[IE] - 0.5 * rho * qq);
    // c = sqrt(c^2) as c^2 * (c^2)^(-1/2); a negative c^2 gives NaN, as sqrt does
    const double c2 = gamma * p * ir;
    const double c = c2 * rsqrt_nr(c2);
    double lam = 0.0;
    for (int d = 0; d < NDIM; ++d) lam += (fabs(u[d]) + c) * inv_dx[d];
    if (isnan(lam) || isnan(rho) || isnan(p)) fl |= 1u;
    if (!(rho > 0.0)) fl |= 2u;
    if (!(p > 0.0)) fl |= 4u;
    return lam;
}

// Wave-speed bound of a cell of a curvilinear 2D grid from its conserved
// state, the unit normals and lengths (nx, ny, len) of its low and high x
// faces (xa, xb) and y faces (ya, yb), and its area: per grid direction, the
// mean of the two faces' area vectors S gives (|u . S| + c |S|) / area.
__host__ __device__ __forceinline__ double curv_cell_lambda(const double* q, double gamma, double gm1,
                                                            const double* xa, const double* xb, const double* ya,
                                                            const double* yb, double area, uint32_t* fl = nullptr) {
    const double ir = 1.0 / q[0];
    const double u = q[1] * ir, v = q[2] * ir;
    const double p = gm1 * (q[3] - 0.5 * q[0] * (u * u + v * v));
    const double c = sqrt(gamma * p * ir);
    double lam = 0.0;
#pragma unroll
    for (int ax = 0; ax < 2; ++ax) {
        const double* a = ax == 0 ? xa : ya;
        const double* b = ax == 0 ? xb : yb;
        const double sx = 0.5 * (a[0] * a[2] + b[0] * b[2]);
        const double sy = 0.5 * (a[1] * a[2] + b[1] * b[2]);
        lam += (fabs(u * sx + v * sy) + c * sqrt(sx * sx + sy * sy)) / area;
    }
    if (fl) {
        // the non-physical flags of cell_lambda: 1 NaN, 2 rho <= 0, 4 p <= 0
        if (isnan(lam) || isnan(q[0]) || isnan(p)) *fl |= 1u;
        if (!(q[0] > 0.0)) *fl |= 2u;
        if (!(p > 0.0)) *fl |= 4u;
    }
    return lam;
}

// ---------------------------------------------------------------------------
// Reverse (adjoint) of the face computation, hand-derived from the forward
// sequence above. The selections of a limiter follow the forward evaluation;
// |x| has derivative 0 at x = 0. The rule LIM is fixed at compile time (0
// minmod, 1 Psi = 1 with kappa = -1, 2 the kappa weights ka, kb, 3 van Leer)
// and the selections are selects: with the scheme tested at run time and the
// limiter's cases as branches, a face took some 700 basic blocks.

// Face states of one variable, with what their reverse needs: the stencil's
// differences and the two limited slopes (mL of the left cell, mR of the right).
template <int LIM>
struct FaceVar {
    double dm, dc, dp, mL, mR;
    __host__ __device__ __forceinline__ void states(const double* q, double ka, double kb, double& qL, double& qR) {
        dm = q[1] - q[0];
        dc = q[2] - q[1];
        dp = q[3] - q[2];
        if (LIM == 2) {
            muscl_kappa_diffs(q[1], q[2], dm, dc, dp, ka, kb, qL, qR);
            mL = mR = 0.0;
        } else {
            mL = LIM == 1 ? dm : (LIM == 3 ? vanleer(dm, dc) : minmod(dm, dc));
            mR = LIM == 1 ? dp : (LIM == 3 ? vanleer(dc, dp) : minmod(dp, dc));
            qL = q[1] + 0.5 * mL;
            qR = q[2] - 0.5 * mR;
        }
    }
    // g[0..3]: dJ/dq of the stencil from qLb = dJ/dQ^L, qRb = dJ/dQ^R.
    __host__ __device__ __forceinline__ void reverse(double qLb, double qRb, double ka, double kb, double* g) const {
        const double hl = 0.5 * qLb, hr = 0.5 * qRb;
        double am, ac, ap;  // dJ/d of the three differences
        if (LIM == 1) {
            am = hl;
            ac = 0.0;
            ap = -hr;
        } else if (LIM == 2) {
            am = ka * qLb;
            ac = kb * (qLb - qRb);
            ap = -ka * qRb;
        } else if (LIM == 3) {
            // d vl(a, b)/da = 2 b^2 / (a + b)^2 and symmetric, zero unless a and b share a sign
            const double sl = dm + dc, sr = dc + dp;
            const bool l = mL != 0.0, r = mR != 0.0;
            const double il = l ? 2.0 / (sl * sl) : 0.0, ir = r ? 2.0 / (sr * sr) : 0.0;
            am = il * dc * dc * hl;
            ac = il * dm * dm * hl - ir * dp * dp * hr;
            ap = -ir * dc * dc * hr;
        } else {
            // the limited slope is one of its two differences or zero; at a tie the
            // derivative follows the limiter as Psi(ratio) x difference, saturating
            // at ratio >= 1: dm for the left state, dc for the right
            const bool ml = mL != 0.0, mr = mR != 0.0;
            const bool lm = mL == dm, rc = mR == dc;
            am = ml && lm ? hl : 0.0;
            ac = (ml && !lm ? hl : 0.0) - (mr && rc ? hr : 0.0);
            ap = mr && !rc ? -hr : 0.0;
        }
        g[0] = -am;
        g[1] = qLb + (am - ac);
        g[2] = qRb + (ac - ap);
        g[3] = ap;
    }
};

__host__ __device__ __forceinline__ double sgn0(double x) { return x > 0.0 ? 1.0 : (x < 0.0 ? -1.0 : 0.0); }

// Reverse of roe_flux<NDIM, AX>: Fb[NV] in, qLb[NV] and qRb[NV] out
// (overwritten). The forward quantities are evaluated as there (the flux
// itself is not needed).
template <int NDIM, int AX>
__host__ __device__ __forceinline__ void roe_flux_vjp(const double* qL, const double* qR, double gm1, const double* Fb,
                                                      double* qLb, double* qRb) {
    constexpr int IE = NDIM + 1;
    const double rL = qL[0], rR = qR[0];
    const double rr = sign_from(rL * rR, rL);
    const double y = rsqrt_nr(rr);
    const double y2 = y * y;
    const double irL = rR * y2, irR = rL * y2;
    const double rt = rr * y;
    const double wR = rR * rcp_nr(rR + rt);
    double uL[NDIM], uR[NDIM], du[NDIM], ut[NDIM];
    double keL = 0.0, keR = 0.0, qqt = 0.0;
#pragma unroll
    for (int d = 0; d < NDIM; ++d) {
        uL[d] = qL[1 + d] * irL;
        uR[d] = qR[1 + d] * irR;
        keL += qL[1 + d] * uL[d];
        keR += qR[1 + d] * uR[d];
        du[d] = uR[d] - uL[d];
        ut[d] = uL[d] + wR * du[d];
        qqt += ut[d] * ut[d];
    }
    const double pL = gm1 * (qL[IE] - 0.5 * keL), pR = gm1 * (qR[IE] - 0.5 * keR);
    const double hL = qL[IE] + pL, hR = qR[IE] + pR;
    const double HL = hL * irL, dH = hR * irR - HL;
    const double Ht = HL + wR * dH;
    const double c2 = gm1 * (Ht - 0.5 * qqt);
    const double rc = rsqrt_nr(c2), c = c2 * rc;
    const double un = ut[AX], aun = fabs(un);
    const bool sub = aun * rc < 1.0;  // subsonic: the acoustic speeds' branch
    const double m = sub ? aun * rc : 1.0, om = 1.0 - m;
    const double sm = copysign(m, un);
    const double dp = pR - pL;
    const double rdu = rt * du[AX];
    const double A = om * rc * dp + sm * rdu;
    const double B = sm * dp + om * c * rdu;
    // ---- reverse, f = Fb / 2 ----
    const double f0 = 0.5 * Fb[0], fE = 0.5 * Fb[IE];
    double f[NDIM], utb[NDIM], uLb[NDIM], uRb[NDIM];
    double fuL = f0, fuR = f0, fut = f0;
    double aunb = -(f0 * (rR - rL) + fE * (qR[IE] - qL[IE]));
    const double mL = qL[1 + AX], mR = qR[1 + AX];
#pragma unroll
    for (int d = 0; d < NDIM; ++d) {
        f[d] = 0.5 * Fb[1 + d];
        fuL += f[d] * uL[d];
        fuR += f[d] * uR[d];
        fut += f[d] * ut[d];
        aunb -= f[d] * (qR[1 + d] - qL[1 + d]);
        utb[d] = -A * f[d];
        uLb[d] = f[d] * mL;
        uRb[d] = f[d] * mR;
    }
    uLb[AX] += fE * hL;
    uRb[AX] += fE * hR;
    // acoustic part
    const double Ab = -(fut + fE * Ht), Bb = -(f[AX] + fE * un);
    const double smb = Ab * rdu + Bb * dp;
    const double tib = Ab * dp, tb = Bb * rdu;
    const double dpb = Ab * om * rc + Bb * sm;
    const double rdub = Ab * sm + Bb * om * c;
    const double omb = sub ? tib * rc + tb * c : 0.0, smu = sub ? smb : 0.0;
    aunb -= omb * rc;
    const double rcb = tib * om - omb * aun + smu * un;
    const double c2b = 0.5 * rc * (tb * om - rcb * rc * rc);
    utb[AX] += smu * rc - B * fE + aunb * sgn0(un);
    const double gc = gm1 * c2b;
    const double Htb = gc - A * fE;
    uLb[AX] -= rdub * rt;
    uRb[AX] += rdub * rt;
    double wRb = Htb * dH;
#pragma unroll
    for (int d = 0; d < NDIM; ++d) {
        const double b = utb[d] - gc * ut[d];
        wRb += b * du[d];
        const double br = wR * b;
        uRb[d] += br;
        uLb[d] += b - br;
    }
    const double HRb = wR * Htb, HLb = Htb - HRb;
    // per side: h = E + p, H = h / rho, p = gm1 (E - m.u / 2), u = m / rho
    const double rtw = rdub * du[AX] * rt, wwb = wRb * wR * (1.0 - wR);
    {
        const double hb = fE * uL[AX] + HLb * irL;
        const double pb = f[AX] - dpb + hb;
        const double keb = -0.5 * gm1 * pb;
        double irb = HLb * hL;
        const double as = aun;
#pragma unroll
        for (int d = 0; d < NDIM; ++d) {
            const double ub = uLb[d] + keb * qL[1 + d];
            irb += ub * qL[1 + d];
            qLb[1 + d] = ub * irL + keb * uL[d] + as * f[d];
        }
        qLb[1 + AX] += fuL;
        qLb[IE] = hb + gm1 * pb + as * fE;
        qLb[0] = irL * (0.5 * (rtw - wwb) - irb * irL) + as * f0;
    }
    {
        const double hb = fE * uR[AX] + HRb * irR;
        const double pb = f[AX] + dpb + hb;
        const double keb = -0.5 * gm1 * pb;
        double irb = HRb * hR;
#pragma unroll
        for (int d = 0; d < NDIM; ++d) {
            const double ub = uRb[d] + keb * qR[1 + d];
            irb += ub * qR[1 + d];
            qRb[1 + d] = ub * irR + keb * uR[d] - aun * f[d];
        }
        qRb[1 + AX] += fuR;
        qRb[IE] = hb + gm1 * pb - aun * fE;
        qRb[0] = irR * (0.5 * (rtw + wwb) - irb * irR) - aun * f0;
    }
}

}  // namespace fvk
