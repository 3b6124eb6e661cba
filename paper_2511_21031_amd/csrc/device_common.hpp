// Device building blocks of the ensemble-averaged RHS stage (gfx950).
//
// Every formula here follows the paper: stiffened-gas liquid (eq. eos_liquid),
// mixture pressure (eq. e:pressure), Keller--Miksis with polytropic or transfer
// contents (eq. keller_miksis, eq. massVaporRate and the contents-pressure
// equation), WENO5 reconstruction and HLLC fluxes (Sec. 3).  The
// arithmetic is arranged for the GPU (one reciprocal per WENO weight set,
// products instead of divisions where the value is unchanged), so results
// agree with a plain evaluation to rounding, not bit for bit.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace bub {

constexpr int NB_MAX = 63;
constexpr double FOUR_PI_3 = 4.18879020478639098461685784437;  // 4 pi / 3
constexpr double FOUR_PI = 12.5663706143591729538505735331;    // 4 pi

// Bubble contents of a context, compiled into the kernels that need them: polytropic gas with the
// general power, polytropic gas with the fifth-root power (3 kappa a whole number of fifths), gas and
// vapour with heat and vapour transfer at the wall (four state fields per bin instead of two), or
// polytropic air (3 kappa = 21/5, the fifth-root power without a branch).
enum Contents : int { CT_POLY = 0, CT_FIFTHS = 1, CT_TRANSFER = 2, CT_AIR = 3 };

// Form of the polytropic power of a kernel (kpow): general, fifth-root, fifth-root for 21/5.
enum PowerForm : int { PW_GENERAL = 0, PW_FIFTHS = 1, PW_AIR = 2 };
__host__ __device__ constexpr int pw_of(int ct) { return ct == CT_AIR ? PW_AIR : ct == CT_FIFTHS ? PW_FIFTHS : PW_GENERAL; }

// Physical constants, passed by value (kernel argument segment -> SGPRs).
struct Phys {
    double gamma, pi_inf, gm1, inv_gm1, gpi;  // gpi = gamma * pi_inf
    double kappa3, sigma2, mu4;               // 3 kappa, 2 sigma, 4 mu
    double p0, rho0;
    int pw_c, pw_d;   // 3 kappa = (5 pw_c - pw_d) / 5 for the fifth-root power (pw_c = 0: the general one)
    // transfer contents (CT_TRANSFER): 3 gamma_b, gas constants, wall temperature and vapour pressure,
    // the heat coefficient (gamma_b - 1)/gamma_b k_b beta_T, D_v beta_c, and the products used below
    double g3, Rg, Rv, T0, pv, kh, betaT, dbc, pvRg, RvT0, inv_RgRv2T0;
};

// Grid: cells per direction, boundary kind per direction (0 periodic,
// 1 reflective, 2 non-reflective; both ends equal), inverse spacing.
struct Grid {
    int n[3];
    int bc[3];
    double inv_dx[3];
    long long N;
};

// Bin table in device memory: r0[nb], w[nb], pg0[nb]; with transfer contents also the equilibrium
// contents pressure pb0[nb], vapour mass mv0[nb] and the gas mass mg[nb] of one bubble of each bin.
struct Bins {
    const double *r0, *w, *pg0;
    const double *pb0, *mv0, *mg;
    int nb;
    int nf;        // state fields per bin: 2 (n R, n Rdot) or 4 (and n p_b, n m_v)
    double m3_eq;  // sum w r0^3
};

// The wave-speed max is gathered in WMAX_SLOTS partial maxima, one per 128-byte line, each
// workgroup posting to slot blockIdx % WMAX_SLOTS: with one counter, the one atomic per wave of
// a large grid (10^5 waves) queues at a single address.
constexpr int WMAX_SLOTS = 64, WMAX_STRIDE = 16;

// Device scalars of one context.
struct Scalars {
    double dt;                // step used by the last rk3_step
    int err_code;             // sticky first error (0 = none)
    int err_bin;
    long long err_cell;
    double t;                 // time at the start of the current step (the stages' clock)
    double t_next;            // time of the state after the last step (the context's clock)
    long long pad_[11];
    // bit patterns of partial maxima of (|u_d| + c)/dx_d (positive doubles order as integers)
    unsigned long long wmax[WMAX_SLOTS * WMAX_STRIDE];
};

// Wavefront max of the CFL wave speed, then one atomic per wave into this workgroup's slot.
__device__ inline void wmax_post(double w, Scalars *sc)
{
    for (int off = 32; off > 0; off >>= 1) {
        const double o = __shfl_xor(w, off, 64);
        w = o > w ? o : w;
    }
    if ((threadIdx.x & 63) == 0 && w > 0.0)
        atomicMax(&sc->wmax[(blockIdx.x % WMAX_SLOTS) * WMAX_STRIDE], (unsigned long long)__double_as_longlong(w));
}

enum { E_NONFINITE = -4, E_NEGR = -5, E_SUBSTEP = -6 };

__device__ inline void raise_error(Scalars *s, int code, long long cell, int bin)
{
    if (atomicCAS(&s->err_code, 0, code) == 0) {
        s->err_cell = cell;
        s->err_bin = bin;
    }
}

// Ghost-cell map of one coordinate.  Periodic: wrap.  Reflective: fold with
// period 2n (one mirror per wall crossing); `flip` toggles on every mirror so
// the normal velocity of the ghost is negated.  Non-reflective (Sec. 5.1, after
// Thompson): the boundary cell itself, so the Riemann problem at the boundary
// face has no jump and no wave enters from outside.
__host__ __device__ inline int map_coord(int i, int n, int bc, bool &flip)
{
    if ((unsigned)i < (unsigned)n) return i;
    if (bc == 0) {
        int m = i % n;
        return m < 0 ? m + n : m;
    }
    if (bc == 2) return i < 0 ? 0 : n - 1;   // non-reflective: the boundary cell's own state
    int p = 2 * n;
    int m = i % p;
    if (m < 0) m += p;
    if (m >= n) {
        m = p - 1 - m;
        flip = !flip;
    }
    return m;
}

// 1/x to full FP64 precision: hardware reciprocal estimate refined by two
// Newton steps (x finite and nonzero).  Cheaper than an IEEE division; agrees
// with 1/x to about one ulp.
__device__ inline double frcp(double x)
{
    double r = __builtin_amdgcn_rcp(x);
    r = fma(fma(-x, r, 1.0), r, r);
    r = fma(fma(-x, r, 1.0), r, r);
    return r;
}

// 1/sqrt(x), x finite and positive: the hardware estimate and one third-order step, about one ulp.
__device__ inline double frsqrt(double x)
{
    const double y = __builtin_amdgcn_rsq(x);
    const double e = fma(-x * y, y, 1.0);
    return fma(y * e, fma(e, 0.375, 0.5), y);
}

// frcp with one Newton step: the estimate is good to about 2^-24, one step leaves at most
// 11 ulp (measured on 4M inputs over 2^+-60; two steps: exact).  For the WENO5 weight sum, whose
// reciprocal scales weights that sum to one.
__device__ inline double frcp1(double x)
{
    double r = __builtin_amdgcn_rcp(x);
    return fma(fma(-x, r, 1.0), r, r);
}

// x^p in FP64 for the polytropic gas pressure (R0/R)^(3 kappa) of a bubble, about 65 vector
// instructions against about 110 for the library power (which carries its logarithm in
// double-double arithmetic).  Textbook reductions (e.g. J.-M. Muller, Elementary Functions,
// 3rd ed., 2016):
//   ln x: x = m 2^e with m in [sqrt(1/2), sqrt(2)); ln m = 2 atanh(s), s = (m-1)/(m+1),
//         |s| < 0.172, by the odd series of atanh up to s^23 (the next term is below 1e-17
//         of the sum); e ln 2 with ln 2 split in a 32-bit head and a tail.  The leading
//         parts (2s and e ln 2) and the product p ln x keep their rounding errors as a
//         second word, so y = p ln x is known to about 2^-60 relative.
//   e^y:  y = k ln 2 + r, |r| <= ln2 / 2, reduced with the same split (Cody and Waite), e^r
//         by its Taylor series up to r^14 (next term below 5e-18), scaled by 2^k.
// Measured against an 80-bit reference: at most 1.2 ulp for x in [e^-160, e^160].
// The series coefficients and constants come from table C (PPOW_TABLE, copied to LDS by the
// caller): as literals the compiler keeps all of them in registers across the caller's loop.
// Zero, infinite, negative or NaN x take the special values of pow.
constexpr int PPOW_N = 28;
constexpr double PPOW_TABLE[PPOW_N] = {
    1.0 / 23.0, 1.0 / 21.0, 1.0 / 19.0, 1.0 / 17.0, 1.0 / 15.0, 1.0 / 13.0, 1.0 / 11.0, 1.0 / 9.0, 1.0 / 7.0,
    1.0 / 5.0, 1.0 / 3.0,                                                  // atanh series, 0..10
    1.0 / 87178291200.0, 1.0 / 6227020800.0, 1.0 / 479001600.0, 1.0 / 39916800.0, 1.0 / 3628800.0,
    1.0 / 362880.0, 1.0 / 40320.0, 1.0 / 5040.0, 1.0 / 720.0, 1.0 / 120.0, 1.0 / 24.0, 1.0 / 6.0,
    0.5,                                                                   // 1/14! .. 1/2!, 11..23
    6.93147180369123816490e-01,   // LN2_HI = 0x3FE62E42FEE00000: k * LN2_HI is exact, 24
    1.90821492927058770002e-10,   // LN2_LO = ln 2 - LN2_HI, 25
    1.44269504088896338700e+00,   // log2(e), 26
    0.70710678118654752440};      // sqrt(1/2), 27

__device__ inline double ppow(double x, double p, const double *__restrict__ C)
{
    // (a class test: x - x == 0 would be contracted into fma(a, b, -x) when x = a * b)
    if (!(x > 0.0) || __builtin_isinf(x)) {
        if (x == 0.0) return p > 0.0 ? 0.0 : (p == 0.0 ? 1.0 : __builtin_huge_val());
        if (x > 0.0) return p > 0.0 ? x : (p == 0.0 ? 1.0 : 0.0);
        return __builtin_nan("");
    }
    int e;
    double m = frexp(x, &e);
    if (m < C[27]) {
        m += m;
        e -= 1;
    }
    // s = f / u with f = m - 1 (exact) and u = m + 1 as a rounded head plus its exact error
    const double f = m - 1.0, u = m + 1.0, ulo = m - (u - 1.0);
    const double iu = frcp(u);
    const double sh = f * iu;
    const double sl = (fma(-sh, u, f) - sh * ulo) * iu;
    const double s2 = sh * sh;
    double t = C[0];
#pragma unroll
    for (int j = 1; j <= 10; ++j) t = fma(t, s2, C[j]);
    // ln x = e LN2_HI + 2 sh + (e LN2_LO + 2 sl + 2 sh^3 t), the first sum kept exactly
    const double fe = (double)e;
    const double a0 = fe * C[24], b0 = 2.0 * sh;
    const double H = a0 + b0;
    const double bb = H - a0;
    const double L = ((a0 - (H - bb)) + (b0 - bb)) + fma(fe, C[25], 2.0 * sl + 2.0 * sh * s2 * t);
    const double lh = H + L, ll = L - (lh - H);
    // y = p ln x as yh + yl
    const double yh = p * lh;
    const double yl = fma(p, lh, -yh) + p * ll;
    const double k = rint(yh * C[26]);
    const double r = (fma(-k, C[24], yh) - k * C[25]) + yl;
    double q = C[11];
#pragma unroll
    for (int j = 12; j <= 23; ++j) q = fma(q, r, C[j]);
    q = fma(q * r, r, r);                     // e^r - 1
    const int ki = (int)fmax(fmin(k, 2100.0), -2100.0);
    return ldexp(1.0 + q, ki);
}

// x^p for p = (5c - d)/5, c >= 1 and 0 <= d <= 4 (the polytropic power 3 kappa of kappa = 1, 1.4, 5/3,
// ...), as x^c z^d with z = x^(-1/5).  z starts from the FP32 hardware log2 / exp2 estimate (relative error
// e below 2e-6 for x in [1e-30, 1e30]) and takes one step of the third-order iteration below, which leaves
// 11 e^3 (below 1e-16) and ends in one rounding; two Newton steps took five operations more and rounded
// twice.  Against an 80-bit reference over x in
// [e^-8, e^8], p = 4.2: at most 5.3 ulp, 1.2 rms (two Newton steps: 8.1 and 2.0; the general power is within
// 1.2 ulp at about four times the instructions).  x must lie in [1e-30, 1e30].
__device__ __forceinline__ double fifth_root_inv(double x)
{
    double z = (double)__builtin_amdgcn_exp2f(-0.2f * __builtin_amdgcn_logf((float)x));
    const double z2 = z * z;
    const double h = fma(x, (z2 * z2) * z, -1.0);   // z = x^(-1/5) (1 + h)^(1/5)
    return fma(z * h, fma(h, 0.12, -0.2), z);       // (1 + h)^(-1/5) = 1 - h/5 + 3 h^2/25 - ...
}

// Air, 3 kappa = 21/5: straight-line powers.
__device__ __forceinline__ double pow_air(double x)
{
    const double z = fifth_root_inv(x);
    const double x2 = x * x, z2 = z * z;
    return ((x2 * x2) * x) * (z2 * z2);
}

__device__ __forceinline__ double pow_fifths(double x, int c, int d)
{
    if (c == 5 && d == 4) return pow_air(x);   // (the branch is uniform)
    const double z = fifth_root_inv(x);
    double xc = 1.0, b = x;
    for (int e = c; e; e >>= 1) {
        if (e & 1) xc *= b;
        b *= b;
    }
    double zd = 1.0;
    for (int k = 0; k < d; ++k) zd *= z;
    return xc * zd;
}

// The polytropic power x^(3 kappa) of a bubble's contents.  PW: the fifth-root form, for contexts whose
// 3 kappa is a whole number of fifths; it needs x in float's normal range and returns NaN for x <= 0 (a
// ratio no admissible state has).  Otherwise ppow (table C in LDS) or, with C null, the library's
// exp2(p log2 x).  The form is a template parameter of the kernels, not a branch: a branch kept both
// forms' registers live through the callers' bin loops (the 2D stage kernel went from 128 to 162 VGPRs
// and lost a wave per SIMD).
template <int PW>
__device__ __forceinline__ double kpow(double x, const Phys &ph, const double *__restrict__ C)
{
    if constexpr (PW == PW_AIR) return pow_air(x);
    else if constexpr (PW == PW_FIFTHS) return pow_fifths(x, ph.pw_c, ph.pw_d);
    else return C ? ppow(x, ph.kappa3, C) : exp2(ph.kappa3 * log2(x));
}

// WENO5-JS face value at the right face of v2 from v0..v4 (cells i-2..i+2), in differences: with
// dk = v(k+1) - vk, the second differences hk = dk - d(k-1) and the one-sided slopes below,
//   4 (beta + eps) = slope^2 + (13/3 h^2 + 4 eps),   face = v2 + sum w r / (6 sum w),
// so the weights' rounding only scales differences of neighbouring cells, and the curvature terms
// 13/3 h^2 + 4 eps belong to a cell, not to a face: both sides of a face share four of them (weno5_pair).
// The nonlinear weights g_k/(eps + beta_k)^2 are normalised through products over the other two
// indicators, so one reciprocal serves all three (the FP64 range holds them; the common factor 4 cancels).
// About 40 FP64 operations per side, 71 per pair (a form in cell values with one indicator after the
// other took 45 and 90; against it the 2D 1024^2 x 31 step went from 2.09 to 2.02 ms, the 3D 256^3 x 21
// split step from 54.6 to 53.1 ms and the Lagrangian step at 192^3 from 3.52 to 3.38 ms).
__device__ __forceinline__ double weno5_curv(double dm, double dp)
{
#pragma clang fp contract(off)
    const double h = dp - dm;
    return fma((13.0 / 3.0) * h, h, 4e-16);
}

__device__ __forceinline__ double weno5_face(double v2, double d0, double d1, double d2, double d3, double c0, double c1,
                                             double c2)
{
#pragma clang fp contract(off)
    const double e0 = fma(3.0, d1, -d0), e1 = d1 + d2, e2 = fma(-3.0, d2, d3);
    double s0 = fma(e0, e0, c0), s1 = fma(e1, e1, c1), s2 = fma(e2, e2, c2);
    s0 *= s0;
    s1 *= s1;
    s2 *= s2;
    // w0 : w1 : w2 = s1 s2 : 6 s0 s2 : 3 s0 s1, on 6 (q_k - v2) = 5 d1 - 2 d0, d1 + 2 d2, 4 d2 - d3
    s0 *= 3.0;
    const double w0 = s1 * s2, h1 = s0 * s2, w2 = s0 * s1, w1 = h1 + h1;
    const double num = fma(w0, fma(2.0, e0, -d1), fma(w1, e1 + d2, w2 * (d2 - e2)));
    return fma(num * (1.0 / 6.0), frcp1((w0 + w2) + w1), v2);
}

__device__ __forceinline__ double weno5(double v0, double v1, double v2, double v3, double v4)
{
    const double d0 = v1 - v0, d1 = v2 - v1, d2 = v3 - v2, d3 = v4 - v3;
    return weno5_face(v2, d0, d1, d2, d3, weno5_curv(d0, d1), weno5_curv(d1, d2), weno5_curv(d2, d3));
}

// Both sides of the face between s[2] and s[3]: bitwise weno5(s0..s4) and weno5(s5..s1).
__device__ __forceinline__ void weno5_pair(const double (&s)[6], double &L, double &R)
{
    const double d0 = s[1] - s[0], d1 = s[2] - s[1], d2 = s[3] - s[2], d3 = s[4] - s[3], d4 = s[5] - s[4];
    const double c1 = weno5_curv(d0, d1), c2 = weno5_curv(d1, d2), c3 = weno5_curv(d2, d3), c4 = weno5_curv(d3, d4);
    L = weno5_face(s[2], d0, d1, d2, d3, c1, c2, c3);
    R = weno5_face(s[3], -d4, -d3, -d2, -d1, c4, c3, c2);
}

// FP32 WENO5-JS for the mixed form: weights normalised through products, as in FP64, on
// indicators rescaled into FP32's range (below), in cell values.  FP32 reciprocals issue at a
// quarter of the rate of other vector instructions, so one reciprocal per
// reconstruction matters here (a ratio form with four took 69 instructions, this
// takes about 52).
__device__ inline float weno5(float v0, float v1, float v2, float v3, float v4)
{
    const float eps = 1e-16f;
    const float c1312 = 13.0f / 12.0f;
    // candidate values: q0 = (2 v0 - 7 v1 + 11 v2)/6, 6 q1 = -v1 + 5 v2 + 2 v3, 3 q2 = (2 v2 + 5 v3 - v4)/2
    float q0 = fmaf(1.0f / 3.0f, v0, fmaf(-7.0f / 6.0f, v1, (11.0f / 6.0f) * v2));
    float q1x6 = fmaf(2.0f, v3, fmaf(5.0f, v2, -v1));
    float q2x3 = fmaf(-0.5f, v4, fmaf(2.5f, v3, v2));
    float d0 = fmaf(-2.0f, v1, v0) + v2, e0 = fmaf(3.0f, v2, fmaf(-4.0f, v1, v0));
    float d1 = fmaf(-2.0f, v2, v1) + v3, e1 = v1 - v3;
    float d2 = fmaf(-2.0f, v3, v2) + v4, e2 = fmaf(-4.0f, v3, fmaf(3.0f, v2, v4));
    float s0 = fmaf(c1312 * d0, d0, fmaf(0.25f * e0, e0, eps));
    float s1 = fmaf(c1312 * d1, d1, fmaf(0.25f * e1, e1, eps));
    float s2 = fmaf(c1312 * d2, d2, fmaf(0.25f * e2, e2, eps));
    // The products of squared indicators leave FP32's range, so each indicator is first divided by
    // the power of two of the smallest (exact: t_i = s_i 2^-e >= 1/2) and held at 2^16 at most: a
    // weight 2^-32 times another is below FP32 resolution, and with t <= 2^16 the products stay
    // below 2^64.  One reciprocal, against one per indicator and one more in a ratio form.
    const int ex = __builtin_amdgcn_frexp_expf(fminf(s0, fminf(s1, s2)));
    float t0 = fminf(__builtin_amdgcn_ldexpf(s0, -ex), 65536.0f);
    float t1 = fminf(__builtin_amdgcn_ldexpf(s1, -ex), 65536.0f);
    float t2 = fminf(__builtin_amdgcn_ldexpf(s2, -ex), 65536.0f);
    t0 *= t0;
    t1 *= t1;
    t2 *= t2;
    // a0 : a1 : a2 = 0.1 t1 t2 : 0.6 t0 t2 : 0.3 t0 t1 = p12 : 6 p02 : 3 p01
    float p12 = t1 * t2, p02 = t0 * t2, p01 = t0 * t1;
    float num = fmaf(p12, q0, fmaf(p02, q1x6, p01 * q2x3));
    float den = fmaf(3.0f, p01, fmaf(6.0f, p02, p12));
    return num * __builtin_amdgcn_rcpf(den);
}

__device__ __forceinline__ void weno5_pair(const float (&s)[6], float &L, float &R)
{
    L = weno5(s[0], s[1], s[2], s[3], s[4]);
    R = weno5(s[5], s[4], s[3], s[2], s[1]);
}

// Reciprocal, square root and division in the reconstruction precision.
__device__ inline double trcp(double x) { return frcp(x); }
__device__ inline float trcp(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ inline double tsqrt(double x) { return sqrt(x); }
__device__ inline float tsqrt(float x) { return __builtin_sqrtf(x); }
__device__ inline double tdiv(double a, double b) { return a / b; }
__device__ inline float tdiv(float a, float b) { return a * __builtin_amdgcn_rcpf(b); }

// Keller--Miksis wall acceleration (eq. keller_miksis) for contents of pressure pb; the R-ddot part of
// d(p_bw)/dt that comes from the viscous term is moved to the left-hand side (exact rearrangement).
// t = (4 mu V + 2 sigma)/R, so p_bw = pb - t; rd = R times the rest of d(p_bw)/dt (the 1/R of that
// derivative cancels: R d(p_bw)/dt = R dp_b/dt + V t).  irho = 1/rho and ic = 1/c of the driving liquid are
// passed in (shared by all bins of a cell).  Its operations are fixed (no contraction), so every kernel that
// takes it gives the same bits; with the 1/R cancelled it is ten operations shorter than the plain form.
__device__ __forceinline__ double km_accel(const Phys &ph, double R, double V, double pb, double rd, double t,
                                           double pinf, double irho, double ic)
{
#pragma clang fp contract(off)
    const double irc = irho * ic, vi = V * ic;
    const double num = fma((1.0 + vi) * ((pb - t) - pinf), irho, fma(rd, irc, -(V * V) * fma(-0.5, vi, 1.5)));
    const double den = fma(R, 1.0 - vi, ph.mu4 * irc);
    return num * frcp(den);
}

// Polytropic contents.  C: the table of the general power (in LDS, or null for the library's).
template <int PW>
__device__ __forceinline__ double km_rddot_t(const Phys &ph, double R, double V, double r0, double pg0, double pinf,
                                             double irho, double ic, const double *__restrict__ C)
{
#pragma clang fp contract(off)
    const double iR = frcp(R);
    const double pb = pg0 * kpow<PW>(r0 * iR, ph, C);
    const double t = fma(ph.mu4, V, ph.sigma2) * iR;
    return km_accel(ph, R, V, pb, V * fma(-ph.kappa3, pb, t), t, pinf, irho, ic);
}

template <int PW>
__device__ __forceinline__ double km_rddot(const Phys &ph, double R, double V, double r0, double pg0, double pinf,
                                           double irho, double ic)
{
    return km_rddot_t<PW>(ph, R, V, r0, pg0, pinf, irho, ic, nullptr);
}

// Transfer contents of one bubble (Sec. 2, eq. massVaporRate and the contents-pressure equation): the
// rates of p_b and m_v for radius R, wall velocity V, pressure p and vapour mass m, gas mass mg.  The
// contents are an ideal-gas mixture at uniform p with mean temperature Tbar = p V_b/(mg Rg + m Rv); the
// wall keeps the liquid temperature T0 with its vapour saturated (partial pressure pv), so with
// S = pv Rg + (p - pv) Rv its vapour mass fraction is chi_w = pv Rg / S and the factor rho_w/(1 - chi_w)
// of the vapour flux is S^2 / (Rg Rv^2 T0 (p - pv)) (rho_w = S/(Rg Rv T0)).  Wall gradients: the transfer
// coefficients times (wall value - bubble mean)/R.
__device__ inline void contents_rates(const Phys &ph, double R, double V, double p, double m, double mg,
                                      double &pdot, double &mdot)
{
#pragma clang fp contract(off)
    const double iR = frcp(R);
    const double Tbar = p * (FOUR_PI_3 * R * R * R) / fma(mg, ph.Rg, m * ph.Rv);
    const double chibar = m / (m + mg);
    const double S = fma(p - ph.pv, ph.Rv, ph.pvRg);
    const double iS = frcp(S);
    const double chiw = ph.pvRg * iS;
    const double flux = ph.dbc * (S * S * ph.inv_RgRv2T0) / (p - ph.pv) * (chiw - chibar) * iR;
    const double dTdr = ph.betaT * (ph.T0 - Tbar) * iR;
    pdot = ph.g3 * iR * fma(-V, p, fma(ph.RvT0, flux, ph.kh * dTdr));
    mdot = FOUR_PI * R * R * flux;
}

// Keller--Miksis wall acceleration for contents of pressure p changing at the rate pdot (transfer contents).
__device__ __forceinline__ double km_rddot_pb(const Phys &ph, double R, double V, double p, double pdot, double pinf,
                                              double irho, double ic)
{
#pragma clang fp contract(off)
    const double t = fma(ph.mu4, V, ph.sigma2) * frcp(R);
    return km_accel(ph, R, V, p, fma(R, pdot, V * t), t, pinf, irho, ic);
}

template <typename T>
__device__ inline T dmin(T a, T b) { return a < b ? a : b; }
template <typename T>
__device__ inline T dmax(T a, T b) { return a > b ? a : b; }

}  // namespace bub
