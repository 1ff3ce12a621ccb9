// fp_device.hpp -- device-side arithmetic of the free-stream-preserving face
// flux for gfx950 (CDNA4, wave64).  Included by the kernel headers only.
//
// One face i+1/2 of one grid line is evaluated by one lane.  The lane reads
// the stencil nodes through a loader (slot r = 0..7 <-> node i-3+r) phase by
// phase, so that only the values of the current phase are live in registers.
// A node comes with its quotients and roots taken (Prim), which the sweeps do
// once per node instead of once per face that uses it:
//   A. cell-face 1/J, metrics and Q~ = Q/J by the central interpolation of
//      the metric order Y; reference state Q* = Q~_f/(1/J)_f and reference
//      face flux F~*_f = F(Q*) s_f                                    [FP64]
//   B. Roe average of nodes i, i+1, unit normal, eigen-structure       [T]
//   C. per stencil node m = i-2..i+3: reference-subtracted dQ~_m, dF~_m
//      [FP64], local Lax-Friedrichs speeds, characteristic projections [T]
//   D. WENO5-JS (or WENO7-JS on slots 0..7) of both split parts of every
//      field, or (linear upwind) the closed form
//      central6(dF~) + (1/60) R Lambda L Delta^5(dQ~)                  [T]
//   E. back-projection and add-back of F~*_f                   [T, FP64 add]
// T is double for the FP64 path and float for the mixed path.
#pragma once
#include <hip/hip_runtime.h>

namespace fpk {

struct SchemeK {
    double gamma;
    double eps;
    int reform;  // 1: reference state subtracted (the paper); 0: standard scheme
    double sg;   // sqrt(gamma)
    double gg;   // gamma / (gamma - 1)
    // floor of the Lax-Friedrichs speeds of the sweep direction (u_n - c,
    // u_n, u_n + c): the face takes max(local speed, floor).  With global
    // speeds the floor is the block's largest local speed, so the face takes
    // the global one (at the face that attains it, the larger of the two
    // roundings); with local speeds it points at zeros.  Never null.
    const double* glf;
};

// ---------------------------------------------------------------------------
// small helpers
// ---------------------------------------------------------------------------

__device__ __forceinline__ float fast_rcp(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ float fast_sqrt(float x) { return __builtin_amdgcn_sqrtf(x); }

// 1/x from the hardware approximation refined by two Newton steps
// (y <- y + y(1 - x y)); within a couple of ulps for normal x.
__device__ __forceinline__ double drcp(double x) {
    double y = __builtin_amdgcn_rcp(x);
    double e = fma(-x, y, 1.0);
    y = fma(y, e, y);
    e = fma(-x, y, 1.0);
    return fma(y, e, y);
}

template <typename T>
__device__ __forceinline__ T rcp(T x);
template <>
__device__ __forceinline__ double rcp<double>(double x) { return drcp(x); }
template <>
__device__ __forceinline__ float rcp<float>(float x) { return fast_rcp(x); }

// Reduced-precision forms for the characteristic basis only (normal,
// tangents, Roe weights, sound speeds, eigenvalue scale): one Newton step
// on the hardware estimate leaves a relative error near 2^-46, far below
// the 1e-12 the flux is held to, and these quantities multiply
// reference-subtracted differences, so the free stream does not see them.
// (Newton's iteration for 1/x and for 1/sqrt(x).)  The reference state keeps
// the two-step drcp.
__device__ __forceinline__ double drcp1(double x) {
    const double y = __builtin_amdgcn_rcp(x);
    return fma(y, fma(-x, y, 1.0), y);
}
__device__ __forceinline__ double drsq1(double x) {
    const double y = __builtin_amdgcn_rsq(x);
    return fma(0.5 * y, fma(-x * y, y, 1.0), y);
}

template <typename T>
__device__ __forceinline__ T rcp1(T x);
template <>
__device__ __forceinline__ double rcp1<double>(double x) { return drcp1(x); }
template <>
__device__ __forceinline__ float rcp1<float>(float x) { return fast_rcp(x); }

template <typename T>
__device__ __forceinline__ T rsq1(T x);
template <>
__device__ __forceinline__ double rsq1<double>(double x) { return drsq1(x); }
template <>
__device__ __forceinline__ float rsq1<float>(float x) { return __builtin_amdgcn_rsqf(x); }

template <typename T>
__device__ __forceinline__ T vsqrt(T x);
template <>
__device__ __forceinline__ double vsqrt<double>(double x) { return sqrt(x); }
template <>
__device__ __forceinline__ float vsqrt<float>(float x) { return fast_sqrt(x); }

// Sums of two products name the one that is fused: left to the compiler, the
// choice varies with the code around, and the sweeps that share the functions
// below must agree (a face's flux is the same number in each of them).
// prod2 = a b + c d with c d rounded.
template <typename T>
__device__ __forceinline__ T prod2(T a, T b, T c, T d) {
    return fma(a, b, c * d);
}

// A node as the faces read it: density, velocity, total energy and, from
// loaders that hold it (LD::CT), the signed thermal speed ct = sign(r) sqrt|r|,
// r = p/rho, so that the sound speed is sqrt(gamma) ct for r > 0, else 0.
// The velocity is rounded once (to_prim), so that rho u is the momentum to the
// last bit or nearly so; energy and pressure see no roots or quotients.  The
// residual's FP64 error is then that of nodes kept as conserved values, or
// lower; with E/rho and rho ct |ct| in their places it was 16 to 42% higher.
template <int DIM>
struct Prim {
    double rho, u[DIM], E, ct;
};

// momentum (a product on its own: contracted into a difference it would keep
// the velocity's rounding) and pressure of a node
template <int DIM>
__device__ __forceinline__ double momentum(const Prim<DIM>& P, int c) {
    return fma(P.rho, P.u[c], 0.0);
}
template <int DIM>
__device__ __forceinline__ double pressure(const Prim<DIM>& P, double gm1) {
    double m2 = 0.0;
#pragma unroll
    for (int c = 0; c < DIM; ++c) m2 = fma(momentum(P, c), P.u[c], m2);
    return gm1 * fma(-0.5, m2, P.E);
}

// sign(x) sqrt|x|: Newton steps on the hardware estimate of 1/sqrt|x| and
// one residual correction (Goldschmidt's form), within a rounding or two
__device__ __forceinline__ double signed_sqrt(double x) {
    const double a = fabs(x);
    double y = __builtin_amdgcn_rsq(a);
    double g = a * y, h = 0.5 * y;
    double r = fma(-h, g, 0.5);
    g = fma(g, r, g);
    h = fma(h, r, h);
    r = fma(-h, g, 0.5);
    g = fma(g, r, g);
    h = fma(h, r, h);
    g = fma(fma(-g, g, a), h, g);
    return a > 0.0 ? copysign(g, x) : 0.0 * x;
}

template <int DIM>
__device__ __forceinline__ void to_prim(const double (&q)[DIM + 2], double gm1, Prim<DIM>& P) {
    const double ir = drcp(q[0]);
    double k2 = 0.0;
    P.rho = q[0];
    P.E = q[DIM + 1];
#pragma unroll
    for (int c = 0; c < DIM; ++c) {
        const double u = q[1 + c] * ir;
        P.u[c] = fma(fma(-q[0], u, q[1 + c]), ir, u);
        k2 = fma(P.u[c], P.u[c], k2);
    }
    P.ct = signed_sqrt(gm1 * fma(P.E, ir, -0.5 * k2));
}

// central face interpolation weights of order Y on slot r (node i in slot 3)
template <int Y>
__device__ __forceinline__ constexpr double iw(int r) {
    if constexpr (Y == 2) {
        return (r == 3 || r == 4) ? 0.5 : 0.0;
    } else if constexpr (Y == 4) {
        return (r == 3 || r == 4) ? 7.0 / 12.0 : ((r == 2 || r == 5) ? -1.0 / 12.0 : 0.0);
    } else if constexpr (Y == 6) {
        return (r == 3 || r == 4) ? 37.0 / 60.0
             : ((r == 2 || r == 5) ? -8.0 / 60.0 : ((r == 1 || r == 6) ? 1.0 / 60.0 : 0.0));
    } else {
        return (r == 3 || r == 4) ? 533.0 / 840.0
             : (r == 2 || r == 5) ? -139.0 / 840.0
             : (r == 1 || r == 6) ? 29.0 / 840.0 : -3.0 / 840.0;
    }
}

// WENO5-JS of a 5-point window a..e (face between c and d, upwind side a),
// in a scaled form.  The window holds twice the split values and eps16 is
// 16 eps: the indicators are evaluated as 4 beta_k = 13/3 t^2 + s^2 of the
// doubled window, i.e. 16 beta_k of the split values, so with 16 eps every
// weight is that of the split values (powers of two: exact), and the
// result is twice their reconstruction.  (The flux splitting's 1/2 is
// applied once, after the back-projection.)  The optimal weights
// C = (1/10, 3/5, 3/10) are folded into the candidates' constants:
// c_k = C_k (6 q_k), and the denominator carries 6 C_k.
// FP64: weights C_k/(beta_k+eps)^2 normalised over one common denominator
// (products of the squared indicators), one reciprocal per reconstruction.
// The window enters through its first differences, the candidates relative to
// c, which comes back at the end: five operations fewer than from the values.
__device__ __forceinline__ double weno5(double a, double b, double c, double d, double e,
                                        double eps16) {
    const double f1 = b - a, f2 = c - b, f3 = d - c, f4 = e - d;
    const double t0 = f2 - f1, t1 = f3 - f2, t2 = f4 - f3;
    const double s0 = fma(3.0, f2, -f1), s1 = f2 + f3, s2 = fma(3.0, f3, -f4);
    const double c0 = fma(0.5, f2, -0.2 * f1), c1 = fma(1.2, f3, 0.6 * f2), c2 = fma(1.2, f3, -0.3 * f4);
    const double k = 13.0 / 3.0;
    double d0 = fma(k * t0, t0, fma(s0, s0, eps16));
    double d1 = fma(k * t1, t1, fma(s1, s1, eps16));
    double d2 = fma(k * t2, t2, fma(s2, s2, eps16));
    d0 *= d0;
    d1 *= d1;
    d2 *= d2;
    const double p0 = d1 * d2, p1 = d0 * d2, p2 = d0 * d1;
    const double num = fma(p0, c0, fma(p1, c1, p2 * c2));
    const double den = fma(p0, 0.6, fma(p1, 3.6, p2 * 1.8));
    return fma(num, drcp1(den), c);
}

// FP32 form: reciprocal weights (no overflow of the products for large beta),
// candidates from the values themselves.  The reference subtraction leaves
// values near zero beside the face, so differences of neighbours are larger
// than c and d and round coarser: the difference form of the FP64 path raises
// the FP32 error of the flux 1.3 to 1.5 times.
__device__ __forceinline__ float weno5(float a, float b, float c, float d, float e, float eps16) {
    const float c0 = fma(1.1f, c, prod2(-0.7f, b, 0.2f, a));
    const float c1 = fma(1.2f, d, prod2(3.0f, c, -0.6f, b));
    const float c2 = fma(-0.3f, e, prod2(1.5f, d, 0.6f, c));
    const float t0 = a - 2.0f * b + c, s0 = a - 4.0f * b + 3.0f * c;
    const float t1 = b - 2.0f * c + d, s1 = d - b;
    const float t2 = c - 2.0f * d + e, s2 = 3.0f * c - 4.0f * d + e;
    const float k = 13.0f / 3.0f;
    const float d0 = fmaf(k * t0, t0, fmaf(s0, s0, eps16));
    const float d1 = fmaf(k * t1, t1, fmaf(s1, s1, eps16));
    const float d2 = fmaf(k * t2, t2, fmaf(s2, s2, eps16));
    const float r0 = fast_rcp(d0 * d0), r1 = fast_rcp(d1 * d1), r2 = fast_rcp(d2 * d2);
    const float num = fmaf(r0, c0, fmaf(r1, c1, r2 * c2));
    const float den = fmaf(r0, 0.6f, fmaf(r1, 3.6f, r2 * 1.8f));
    return fma(num, fast_rcp(den), 0.0f);
}

// The reconstructions below take twice the split values; their indicators
// are quadratic, so eps enters scaled and the weights are those of the split
// values (powers of two: exact), the result twice their reconstruction.
//
// Indicators and weights see the window through its first differences f_j.
// The candidates do too in FP64 (relative to the value beside the face, which
// comes back at the end), but use the values themselves in FP32: the
// reference subtraction leaves values near zero there, and rounding the
// larger differences would cost accuracy.
//
// FP64 forms the weights over one common denominator, so that a
// reconstruction takes two reciprocals (each a quarter-rate instruction and
// four Newton operations) instead of five or six.  The weights depend on the
// indicators' ratios alone, and products of six (five) indicators would
// leave the range of FP64 from indicators of 1e51 (1e61): each window's
// indicators are first brought to order one by a power of two, which rounds
// nothing.  What is added to them then is 1e-50 (1e-60) of the largest, below
// its rounding, and keeps the products off zero for any eps.
// FP32 has no such range and takes a reciprocal per indicator.
// RK3 steps with the indicators in values and a reciprocal each, and now:
// FP64 WENOCU6 145x113x97 1.55 and 1.29 ms (1.25 without the power of two),
// FP32-mixed WENO7-M8 191x161x133 2.84 and 2.65 ms.

// 2^-k for x in [2^k, 2^(k+1)), x > 0
__device__ __forceinline__ double pow2_rcp(double x) {
    const unsigned long long e = __builtin_bit_cast(unsigned long long, x) >> 52 & 0x7ff;
    return __builtin_bit_cast(double, (0x7feull - e) << 52);
}

// one indicator of WENO7: a quadratic form in three consecutive differences
template <typename T>
__device__ __forceinline__ T form3(T f1, T f2, T f3, T c11, T c12, T c13, T c22, T c23, T c33, T eps) {
    return fma(f1, fma(c13, f3, prod2(c12, f2, c11, f1)), fma(f2, prod2(c23, f3, c22, f2), fma(c33 * f3, f3, eps)));
}

// WENO7-JS of a 7-point window v[0..6] (face between v[3] and v[4], upwind
// side v[0]): four cubic candidates, optimal weights (1, 12, 18, 4)/35,
// smoothness indicators as the integer quadratic forms (240 x the Jiang-Shu
// measure; in differences their coefficients are a quarter to a half as
// large), weights C_k/(beta_k+eps)^2.  Takes 4 eps.
template <typename T>
__device__ __forceinline__ T weno7(const T (&v)[7], T eps) {
    const T a = v[0], b = v[1], c = v[2], d = v[3], e = v[4], f = v[5], g = v[6];
    const T f0 = b - a, f1 = c - b, f2 = d - c, f3 = e - d, f4 = f - e, f5 = g - f;
    constexpr bool F64 = sizeof(T) == 8;
    T b0 = form3<T>(f0, f1, f2, T(547), T(-2788), T(1854), T(3708), T(-5188), T(2107), eps);
    T b1 = form3<T>(f1, f2, f3, T(267), T(-1108), T(494), T(1468), T(-1428), T(547), eps);
    T b2 = form3<T>(f2, f3, f4, T(547), T(-1428), T(494), T(1468), T(-1108), T(267), eps);
    T b3 = form3<T>(f3, f4, f5, T(2107), T(-5188), T(1854), T(3708), T(-2788), T(547), eps);
    if constexpr (F64) {
        // b0 + b3 sees all six differences: b1 and b2 are below 6 times it
        const T sc = pow2_rcp(b0 + b3), lo = T(1e-50);
        b0 = fma(b0, sc, lo);
        b1 = fma(b1, sc, lo);
        b2 = fma(b2, sc, lo);
        b3 = fma(b3, sc, lo);
    }
    b0 *= b0;
    b1 *= b1;
    b2 *= b2;
    b3 *= b3;
    if constexpr (F64) {
        const T b01 = b0 * b1, b23 = b2 * b3;
        const T a0 = b1 * b23, a1 = b0 * (T(12) * b23), a2 = b3 * (T(18) * b01), a3 = b2 * (T(4) * b01);
        const T q0 = fma(T(13), f2, prod2(T(-10), f1, T(3), f0));  // 12 (q_k - d)
        const T q1 = prod2(T(3), f3, T(4), f2) - f1;
        const T q2 = T(6) * f3 + f2 - f4;
        const T q3 = prod2(T(-4), f4, T(9), f3) + f5;
        const T num = fma(a3, q3, fma(a2, q2, prod2(a1, q1, a0, q0)));
        return fma(num, rcp<T>(T(12) * (a0 + a1 + a2 + a3)), d);
    } else {
        const T q0 = fma(T(25), d, fma(T(-23), c, prod2(T(13), b, T(-3), a)));
        const T q1 = b - T(5) * c + T(13) * d + T(3) * e;
        const T q2 = -c + T(7) * d + T(7) * e - f;
        const T q3 = fma(T(-5), f, prod2(T(13), e, T(3), d)) + g;
        const T a0 = rcp<T>(b0), a1 = T(12) * rcp<T>(b1), a2 = T(18) * rcp<T>(b2), a3 = T(4) * rcp<T>(b3);
        const T num = fma(a3, q3, fma(a2, q2, prod2(a1, q1, a0, q0)));
        return fma(num, rcp<T>(T(12) * (a0 + a1 + a2 + a3)), T(0));
    }
}

// WENOCU6 (the adaptive central-upwind sixth-order WENO of Hu, Wang and Adams,
// Remark 2) of a 6-point window v[0..5] = f_{i-2} .. f_{i+3}, the face between
// v[2] and v[3].  Candidates: the three upwind quadratics of WENO5 and the
// downwind one on {i+1, i+2, i+3}; optimal weights (1, 9, 9, 1)/20 (the
// sixth-order central interpolation).  The downwind slot's indicator is beta6,
// the Jiang-Shu measure (derivative orders 1..5 over cell i) of the quintic
// through all six cell averages, evaluated from the quintic's Taylor
// coefficients D_l = p^(l) at the centre of cell i, which are combinations of
// the window's first to fifth differences (f, t, u; D4, D5 are the centred
// fourth and the fifth difference): beta6 keeps its accuracy in FP32, where
// the expanded integer quadratic form of the six values cancels to noise.
// Every indicator is formed times four (4 beta_k = 13/3 t^2 + s^2), so this
// takes 16 eps.  Weights alpha_k = d_k (C + tau6/(beta_k + eps))^2, C = 20,
// tau6 = beta6 - (beta_0 + 4 beta_1 + beta_2)/6, evaluated as
// ((C m + tau6 m/(beta_k+eps)) / (m + |tau6|))^2 with m = min_k (beta_k+eps):
// the same ratios, every factor in [-C, C].
template <typename T>
__device__ __forceinline__ T wenocu6(const T (&v)[6], T eps) {
    const T a = v[0], b = v[1], c = v[2], d = v[3], e = v[4], f = v[5];
    const T f1 = b - a, f2 = c - b, f3 = d - c, f4 = e - d, f5 = f - e;
    const T t0 = f2 - f1, t1 = f3 - f2, t2 = f4 - f3, t3 = f5 - f4;
    const T u1 = t1 - t0, u2 = t2 - t1, u3 = t3 - t2;
    const T s0 = T(3) * f2 - f1, s1 = f2 + f3, s2 = T(3) * f3 - f4;
    const T k13 = T(13.0 / 3.0);
    constexpr bool F64 = sizeof(T) == 8;
    const T b0 = prod2(s0, s0, k13 * t0, t0);
    const T b1 = prod2(s1, s1, k13 * t1, t1);
    const T b2 = prod2(s2, s2, k13 * t2, t2);
    const T D4 = u2 - u1, D5 = (u3 - u2) - D4;
    const T G1 = s1 - T(341.0 / 2880.0) * u1 - T(1118.0 / 2880.0) * u2 + T(259.0 / 2880.0) * u3;  // 2 D1
    const T G2 = prod2(T(-0.25), D4, T(2), t1);                                                        // 2 D2
    const T G3 = fma(T(-7.0 / 12.0), u3, prod2(T(26.0 / 12.0), u2, T(5.0 / 12.0), u1));  // 2 D3
    const T h1 = G1 + G3 * T(1.0 / 12.0) + D5 * T(1.0 / 480.0);
    const T h2 = prod2(D4, T(7.0 / 40.0), G2, T(13.0 / 12.0));
    const T h3 = prod2(D5, T(4709.0 / 26880.0), G3, T(1043.0 / 960.0));
    const T b6 = fma(D5 * D5, T(50467427.0 / 11612160.0),
                     fma(D4 * D4, T(87617.0 / 20160.0), fma(G3, h3, prod2(G2, h2, G1, h1))));
    T tau = b6 - (b0 + T(4) * b1 + b2) * T(1.0 / 6.0);
    T e0, e1, e2, e3;
    if constexpr (F64) {
        // beta6 sees all five differences: the others are below 3 times it
        const T sc = pow2_rcp(b6 + eps), es = fma(eps, sc, T(1e-60));
        tau *= sc;
        e0 = fma(b0, sc, es);
        e1 = fma(b1, sc, es);
        e2 = fma(b2, sc, es);
        e3 = fma(b6, sc, es);
    } else {
        e0 = b0 + eps;
        e1 = b1 + eps;
        e2 = b2 + eps;
        e3 = b6 + eps;
    }
    const T m = fmin(fmin(e0, e1), fmin(e2, e3));
    const T mt = m + fabs(tau);
    if constexpr (F64) {
        const T e01 = e0 * e1, e23 = e2 * e3, P = e01 * e23;
        const T R = rcp<T>(P * mt), ig = P * R;  // 1/(m + |tau|)
        const T sC = T(20) * (m * ig);
        const T x = tau * m * ig * (mt * R);  // tau m / ((m + |tau|) e0 e1 e2 e3)
        const T x01 = x * e23, x23 = x * e01;
        const T w0 = fma(x01, e1, sC), w1 = fma(x01, e0, sC), w2 = fma(x23, e3, sC), w3 = fma(x23, e2, sC);
        const T a0 = w0 * w0, a1 = T(9) * (w1 * w1), a2 = T(9) * (w2 * w2), a3 = w3 * w3;
        const T q0 = prod2(T(-2), f1, T(5), f2), q1 = T(2) * f3 + f2;  // 6 (q_k - c)
        const T q2 = T(4) * f3 - f4, q3 = fma(T(2), f5, prod2(T(-5), f4, T(6), f3));
        const T num = fma(a3, q3, fma(a2, q2, prod2(a1, q1, a0, q0)));
        return fma(num, rcp<T>(T(6) * (a0 + a1 + a2 + a3)), c);
    } else {
        const T ig = rcp<T>(mt);
        const T sC = T(20) * (m * ig), st = tau * ig;
        const T w0 = fma(st, m * rcp<T>(e0), sC), w1 = fma(st, m * rcp<T>(e1), sC);
        const T w2 = fma(st, m * rcp<T>(e2), sC), w3 = fma(st, m * rcp<T>(e3), sC);
        const T a0 = w0 * w0, a1 = T(9) * (w1 * w1), a2 = T(9) * (w2 * w2), a3 = w3 * w3;
        const T q0 = fma(T(11), c, prod2(T(-7), b, T(2), a));
        const T q1 = -b + T(5) * c + T(2) * d;
        const T q2 = prod2(T(5), d, T(2), c) - e;
        const T q3 = fma(T(2), f, prod2(T(-7), e, T(11), d));
        const T num = fma(a3, q3, fma(a2, q2, prod2(a1, q1, a0, q0)));
        return fma(num, rcp<T>(T(6) * (a0 + a1 + a2 + a3)), T(0));
    }
}

// ---------------------------------------------------------------------------
// phase A: cell-face reference state
// ---------------------------------------------------------------------------

template <int DIM>
struct FaceRef {
    double Vf;
    double sf[DIM];
    double Qs[DIM + 2];  // Q* (zero for the standard scheme)
    double us[DIM];      // u*
    double ps;           // p*
    double Fts[DIM + 2]; // F(Q*) . s_f
    double s2;           // |s_f|^2
};

template <int DIM, int Y, class LD>
__device__ __forceinline__ void face_ref(const LD& ld, const SchemeK& sk, FaceRef<DIM>& R) {
    constexpr int NV = DIM + 2, E = NV - 1;
    constexpr int r0 = 4 - Y / 2, r1 = 4 + Y / 2;  // interpolation slots [r0, r1)
    double Vf = 0.0, sf[DIM], Qt[NV];
#pragma unroll
    for (int c = 0; c < DIM; ++c) sf[c] = 0.0;
#pragma unroll
    for (int v = 0; v < NV; ++v) Qt[v] = 0.0;
#pragma unroll
    for (int r = r0; r < r1; ++r) ld.interp(r, iw<Y>(r), Qt, Vf, sf);
    R.Vf = Vf;
#pragma unroll
    for (int c = 0; c < DIM; ++c) R.sf[c] = sf[c];
    R.ps = 0.0;
#pragma unroll
    for (int v = 0; v < NV; ++v) R.Qs[v] = 0.0;
#pragma unroll
    for (int c = 0; c < DIM; ++c) R.us[c] = 0.0;
    if (sk.reform) {
        const double iVf = drcp(Vf);
#pragma unroll
        for (int v = 0; v < NV; ++v) R.Qs[v] = Qt[v] * iVf;
        const double irs = drcp(R.Qs[0]);
        double m2 = 0.0;
#pragma unroll
        for (int c = 0; c < DIM; ++c) {
            R.us[c] = R.Qs[1 + c] * irs;
            m2 += R.Qs[1 + c] * R.us[c];
        }
        R.ps = (sk.gamma - 1.0) * (R.Qs[E] - 0.5 * m2);
    }
    double U = 0.0, s2 = 0.0;
#pragma unroll
    for (int c = 0; c < DIM; ++c) {
        U += R.us[c] * sf[c];
        s2 += sf[c] * sf[c];
    }
    R.Fts[0] = R.Qs[0] * U;
#pragma unroll
    for (int c = 0; c < DIM; ++c) R.Fts[1 + c] = prod2(R.ps, sf[c], R.Qs[1 + c], U);
    R.Fts[E] = (R.Qs[E] + R.ps) * U;
    R.s2 = s2;
}

// ---------------------------------------------------------------------------
// phase B: Roe average and characteristic basis
// ---------------------------------------------------------------------------

template <int DIM, typename T>
struct Eig {
    T n[DIM], uh[DIM], t1[DIM], t2[3];
    T un, Hh, ch, hq2, ut1, ut2, sigma;
    // the projection's scales, halved: with b2 = (gamma-1)/c^2 and ic = 1/c,
    // pB = b2/2 and pI = ic/2
    T pB, pI;
};

template <int DIM, typename T, class LD>
__device__ __forceinline__ void roe(const LD& ld, const SchemeK& sk, const FaceRef<DIM>& R,
                                    Eig<DIM, T>& S) {
    const double gm1 = sk.gamma - 1.0;
    const double isn = drsq1(R.s2);  // 1/|s_f|
#pragma unroll
    for (int c = 0; c < DIM; ++c) S.n[c] = T(R.sf[c] * isn);
    S.sigma = T(R.s2 * isn * drcp1(R.Vf));
    Prim<DIM> L, Q;
    ld.prim(3, L);
    ld.prim(4, Q);
    // H = |u|^2/2 + gamma/(gamma - 1) p/rho
    auto enthalpy = [&](const Prim<DIM>& P) {
        if constexpr (LD::CT) {
            double k2 = 0.0;
#pragma unroll
            for (int c = 0; c < DIM; ++c) k2 = fma(P.u[c], P.u[c], k2);
            return fma(sk.gg * P.ct, fabs(P.ct), 0.5 * k2);
        } else {
            return (P.E + pressure(P, gm1)) * drcp(P.rho);
        }
    };
    const double HL = enthalpy(L), HR = enthalpy(Q);
    const T wL = T(L.rho) * rsq1<T>(T(L.rho)), wR = T(Q.rho) * rsq1<T>(T(Q.rho));
    const T iwr = rcp1<T>(wL + wR);
    T q2 = T(0), un = T(0);
#pragma unroll
    for (int c = 0; c < DIM; ++c) {
        S.uh[c] = prod2(wR, T(Q.u[c]), wL, T(L.u[c])) * iwr;
        q2 += S.uh[c] * S.uh[c];
        un += S.uh[c] * S.n[c];
    }
    S.un = un;
    S.Hh = prod2(wR, T(HR), wL, T(HL)) * iwr;
    const T c2 = T(gm1) * fma(T(-0.5), q2, S.Hh);
    const T ic = rsq1<T>(c2);
    S.ch = c2 * ic;
    S.hq2 = T(0.5) * q2;
    S.pB = T(0.5 * gm1) * (ic * ic);
    S.pI = T(0.5) * ic;
    if constexpr (DIM == 2) {
        S.t1[0] = -S.n[1];
        S.t1[1] = S.n[0];
        S.ut1 = prod2(S.uh[1], S.t1[1], S.uh[0], S.t1[0]);
        S.ut2 = T(0);
    } else {
        // a = argmin |n_k|, components within 1e-10 count as tied and the
        // lowest k wins; t1 = normalize(n x e_a), t2 = n x t1
        const T tie = T(1e-10);
        const T a0 = fabs(S.n[0]), a1 = fabs(S.n[1]), a2 = fabs(S.n[2]);
        int a = 0;
        T am = a0;
        if (a1 < am - tie) { a = 1; am = a1; }
        if (a2 < am - tie) { a = 2; }
        T x0, x1, x2;
        if (a == 0) { x0 = T(0); x1 = S.n[2]; x2 = -S.n[1]; }
        else if (a == 1) { x0 = -S.n[2]; x1 = T(0); x2 = S.n[0]; }
        else { x0 = S.n[1]; x1 = -S.n[0]; x2 = T(0); }
        const T ix = rsq1<T>(fma(x2, x2, prod2(x1, x1, x0, x0)));
        S.t1[0] = x0 * ix;
        S.t1[1] = x1 * ix;
        S.t1[2] = x2 * ix;
        S.t2[0] = prod2(S.n[1], S.t1[2], -S.n[2], S.t1[1]);
        S.t2[1] = prod2(S.n[2], S.t1[0], -S.n[0], S.t1[2]);
        S.t2[2] = prod2(S.n[0], S.t1[1], -S.n[1], S.t1[0]);
        S.ut1 = fma(S.uh[2], S.t1[2], prod2(S.uh[1], S.t1[1], S.uh[0], S.t1[0]));
        S.ut2 = fma(S.uh[2], S.t2[2], prod2(S.uh[1], S.t2[1], S.uh[0], S.t2[0]));
    }
}

// ---------------------------------------------------------------------------
// phase C helper: reference-subtracted values and LF speeds at one node
// ---------------------------------------------------------------------------

// n.u and the sound speed of a node of pressure p
template <int DIM, typename T, bool CT>
__device__ __forceinline__ void node_speeds(const SchemeK& sk, const Eig<DIM, T>& S, const Prim<DIM>& P, double p,
                                            T& un, T& cs) {
    un = T(0);
#pragma unroll
    for (int c = 0; c < DIM; ++c) un += S.n[c] * T(P.u[c]);
    if constexpr (CT) {
        cs = T(sk.sg) * fmax(T(P.ct), T(0));
    } else {
        const T c2 = T(sk.gamma * p) * rcp1<T>(T(P.rho));
        cs = c2 > T(0) ? c2 * rsq1<T>(c2) : T(0);
    }
}

template <int DIM, typename T>
struct NodeDiff {
    double dQ[DIM + 2], dF[DIM + 2];
    T un, cs;
};

template <int DIM, typename T, class LD>
__device__ __forceinline__ void node_diff(const LD& ld, int r, const SchemeK& sk,
                                          const FaceRef<DIM>& R, const Eig<DIM, T>& S,
                                          NodeDiff<DIM, T>& N) {
    constexpr int NV = DIM + 2, E = NV - 1;
    Prim<DIM> P;
    double V, s[DIM];
    ld.prim(r, P);
    ld.metric(r, V, s);
    double U = 0.0, Us = 0.0;
#pragma unroll
    for (int c = 0; c < DIM; ++c) {
        U += P.u[c] * s[c];
        Us += R.us[c] * s[c];
    }
    const double p = pressure(P, sk.gamma - 1.0);
    const double dp = p - R.ps;
    N.dF[0] = prod2(P.rho, U, -R.Qs[0], Us);
    N.dQ[0] = (P.rho - R.Qs[0]) * V;
#pragma unroll
    for (int c = 0; c < DIM; ++c) {
        const double m = momentum(P, c);
        N.dF[1 + c] = fma(dp, s[c], prod2(m, U, -R.Qs[1 + c], Us));
        N.dQ[1 + c] = (m - R.Qs[1 + c]) * V;
    }
    N.dF[E] = prod2(P.E + p, U, -(R.Qs[E] + R.ps), Us);
    N.dQ[E] = (P.E - R.Qs[E]) * V;
    node_speeds<DIM, T, LD::CT>(sk, S, P, p, N.un, N.cs);
}

// l_s . w for the five (four in 2D) fields, using the structure of the Euler
// eigenvectors: l_0 w = (phi - psi)/2, l_1 w = w_0 - phi, l_t w = t.w_m -
// (u.t) w_0, l_E w = (phi + psi)/2 with phi = b2 (|u|^2/2 w_0 - u.w_m + w_E)
// and psi = (n.w_m - u_n w_0)/c; evaluated as phi/2 and psi/2 with the
// halved scales of Eig.
template <int DIM, typename T>
__device__ __forceinline__ void project(const Eig<DIM, T>& S, const T (&w)[DIM + 2],
                                        T (&a)[DIM + 2]) {
    constexpr int E = DIM + 1;
    T uw = T(0), nw = T(0), t1w = T(0), t2w = T(0);
#pragma unroll
    for (int c = 0; c < DIM; ++c) {
        uw += S.uh[c] * w[1 + c];
        nw += S.n[c] * w[1 + c];
        t1w += S.t1[c] * w[1 + c];
        if constexpr (DIM == 3) t2w += S.t2[c] * w[1 + c];
    }
    const T phi = S.pB * (S.hq2 * w[0] - uw + w[E]);
    const T nu = nw - S.un * w[0];  // psi = nu pI
    a[0] = fma(-nu, S.pI, phi);
    a[1] = fma(T(-2), phi, w[0]);
    a[2] = t1w - S.ut1 * w[0];
    if constexpr (DIM == 3) a[3] = t2w - S.ut2 * w[0];
    a[E] = fma(nu, S.pI, phi);
}

// R h: back to conservative components
template <int DIM, typename T>
__device__ __forceinline__ void backproject(const Eig<DIM, T>& S, const T (&h)[DIM + 2],
                                            T (&o)[DIM + 2]) {
    constexpr int E = DIM + 1;
    const T h0 = h[0], h1 = h[1], hE = h[E];
    const T hsum = h0 + h1 + hE, hdif = hE - h0;
    o[0] = hsum;
#pragma unroll
    for (int c = 0; c < DIM; ++c) {
        T m = fma(S.t1[c], h[2], prod2(S.ch * S.n[c], hdif, S.uh[c], hsum));
        if constexpr (DIM == 3) m = fma(S.t2[c], h[3], m);
        o[1 + c] = m;
    }
    T en = fma(S.ut1, h[2], fma(S.hq2, h1, prod2(S.ch * S.un, hdif, S.Hh, h0 + hE)));
    if constexpr (DIM == 3) en = fma(S.ut2, h[3], en);
    o[E] = en;
}

// ---------------------------------------------------------------------------
// the face flux: WENO5-JS and WENOCU6 (stencil nodes i-2 .. i+3, slots 1..6)
// ---------------------------------------------------------------------------

template <int DIM, int Y, typename T, bool CU6, class LD>
__device__ __forceinline__ void face_flux_weno(const LD& ld, const SchemeK& sk,
                                               double (&Fo)[DIM + 2]) {
    constexpr int NV = DIM + 2, E = NV - 1;
    FaceRef<DIM> R;
    face_ref<DIM, Y>(ld, sk, R);
    Eig<DIM, T> S;
    roe<DIM, T>(ld.after(R.Vf), sk, R, S);
    // per stencil node: projections of dF~ (a) and dQ~ (b) on every field
    T a[NV][6], b[NV][6];
    T mxm = T(0), mx0 = T(0), mxp = T(0);
    double chain = double(S.pI);
#pragma unroll
    for (int r = 1; r <= 6; ++r) {
        NodeDiff<DIM, T> N;
        node_diff<DIM, T>(ld.after(chain), r, sk, R, S, N);
        chain = N.dQ[0];
        mxm = fmax(mxm, fabs(N.un - N.cs));
        mx0 = fmax(mx0, fabs(N.un));
        mxp = fmax(mxp, fabs(N.un + N.cs));
        T w[NV], pa[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v) w[v] = T(N.dF[v]);
        project<DIM, T>(S, w, pa);
#pragma unroll
        for (int v = 0; v < NV; ++v) a[v][r - 1] = pa[v];
#pragma unroll
        for (int v = 0; v < NV; ++v) w[v] = T(N.dQ[v]);
        project<DIM, T>(S, w, pa);
#pragma unroll
        for (int v = 0; v < NV; ++v) b[v][r - 1] = pa[v];
    }
    // LF speeds: fields (u_n - c), (u_n) x (DIM - 1), (u_n + c)
    T lam[NV];
    lam[0] = fmax(S.sigma * mxm, T(sk.glf[0]));
    const T l1 = fmax(S.sigma * mx0, T(sk.glf[1]));
#pragma unroll
    for (int v = 1; v < E; ++v) lam[v] = l1;
    lam[E] = fmax(S.sigma * mxp, T(sk.glf[2]));
    // WENOCU6's eps may be far below the FP32 normal range (1e-40 in the
    // published scheme): the FP32 path floors it at 1e-30.  The
    // reconstructions take twice the split values a +- lambda b (the split's
    // 1/2 goes on the back-projected sum) and scale their indicators by 4:
    // 16 eps.
    const T eps = (CU6 && sizeof(T) == 4) ? fmax(T(sk.eps), T(1e-30)) : T(sk.eps);
    const T epsw = T(16) * eps;
    T h[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        T vp[6], vm[6];
#pragma unroll
        for (int r = 0; r < 6; ++r) {
            vp[r] = a[v][r] + lam[v] * b[v][r];
            vm[r] = a[v][5 - r] - lam[v] * b[v][5 - r];
        }
        if constexpr (CU6)
            h[v] = wenocu6<T>(vp, epsw) + wenocu6<T>(vm, epsw);
        else
            h[v] = weno5(vp[0], vp[1], vp[2], vp[3], vp[4], epsw) +
                   weno5(vm[0], vm[1], vm[2], vm[3], vm[4], epsw);
    }
    T o[NV];
    backproject<DIM, T>(S, h, o);
#pragma unroll
    for (int v = 0; v < NV; ++v) Fo[v] = fma(0.5, double(o[v]), R.Fts[v]);
}

// ---------------------------------------------------------------------------
// the face flux: WENO7-JS (Remark 2), stencil nodes i-3 .. i+4 (slots 0..7)
// ---------------------------------------------------------------------------

template <int DIM, int Y, typename T, class LD>
__device__ __forceinline__ void face_flux_weno7(const LD& ld, const SchemeK& sk,
                                                double (&Fo)[DIM + 2]) {
    constexpr int NV = DIM + 2, E = NV - 1;
    FaceRef<DIM> R;
    face_ref<DIM, Y>(ld, sk, R);
    Eig<DIM, T> S;
    roe<DIM, T>(ld.after(R.Vf), sk, R, S);
    T a[NV][8], b[NV][8];
    T mxm = T(0), mx0 = T(0), mxp = T(0);
    double chain = double(S.pI);
#pragma unroll
    for (int r = 0; r <= 7; ++r) {
        NodeDiff<DIM, T> N;
        node_diff<DIM, T>(ld.after(chain), r, sk, R, S, N);
        chain = N.dQ[0];
        mxm = fmax(mxm, fabs(N.un - N.cs));
        mx0 = fmax(mx0, fabs(N.un));
        mxp = fmax(mxp, fabs(N.un + N.cs));
        T w[NV], pa[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v) w[v] = T(N.dF[v]);
        project<DIM, T>(S, w, pa);
#pragma unroll
        for (int v = 0; v < NV; ++v) a[v][r] = pa[v];
#pragma unroll
        for (int v = 0; v < NV; ++v) w[v] = T(N.dQ[v]);
        project<DIM, T>(S, w, pa);
#pragma unroll
        for (int v = 0; v < NV; ++v) b[v][r] = pa[v];
    }
    T lam[NV];
    lam[0] = fmax(S.sigma * mxm, T(sk.glf[0]));
    const T l1 = fmax(S.sigma * mx0, T(sk.glf[1]));
#pragma unroll
    for (int v = 1; v < E; ++v) lam[v] = l1;
    lam[E] = fmax(S.sigma * mxp, T(sk.glf[2]));
    // twice the split values, 4 eps; the split's 1/2 on the back-projected sum
    const T eps4 = T(4) * T(sk.eps);
    T h[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        T vp[7], vm[7];
#pragma unroll
        for (int r = 0; r < 7; ++r) {
            vp[r] = a[v][r] + lam[v] * b[v][r];
            vm[r] = a[v][7 - r] - lam[v] * b[v][7 - r];
        }
        h[v] = weno7<T>(vp, eps4) + weno7<T>(vm, eps4);
    }
    T o[NV];
    backproject<DIM, T>(S, h, o);
#pragma unroll
    for (int v = 0; v < NV; ++v) Fo[v] = fma(0.5, double(o[v]), R.Fts[v]);
}

// ---------------------------------------------------------------------------
// the face flux: fifth-order linear upwind
// ---------------------------------------------------------------------------
// With the optimal weights the two split parts reconstruct linearly, and
// since (LU5+ + LU5-)/2 is the sixth-order central interpolation and
// (LU5+ - LU5-)/2 the fifth difference (1,-5,10,-10,5,-1)/60,
//   sum_s r_s (h+_s + h-_s) = central6(dF~) + (1/60) R Lambda L Delta^5(dQ~),
// which is the linear-upwind member of eq. new_form_linear_upwind.

// The central sum is linear in the node fluxes, so the reference flux leaves
// it as one term per face: central6(dF~) = central6(F~) - F(Q*).s6 with
// s6 = central6(s).  With the add-back F(Q*).s_f the flux keeps
// F(Q*).(s_f - s6), which vanishes for sixth-order metrics, whose
// interpolation is central6 itself; s_f - s6 is summed from the difference of
// the weights, free of the rounding of two sums.  The pressure takes p - p*
// node by node, and the whole p* s_f at the face: at low Mach numbers its
// rounding would be the flux's largest.  (The fifth difference takes Q - Q*
// node by node: its weights would amplify the rounding of Q.)

template <int DIM, int Y, typename T, class LD>
__device__ __forceinline__ void face_flux_lu5(const LD& ld, const SchemeK& sk,
                                              double (&Fo)[DIM + 2]) {
    constexpr int NV = DIM + 2, E = NV - 1;
    constexpr double c6[6] = {1.0 / 60, -8.0 / 60, 37.0 / 60, 37.0 / 60, -8.0 / 60, 1.0 / 60};
    constexpr double d5[6] = {1.0, -5.0, 10.0, -10.0, 5.0, -1.0};
    // weights of s_f - s6 on slots 1..6
    constexpr double df[6] = {iw<Y>(1) - c6[0], iw<Y>(2) - c6[1], iw<Y>(3) - c6[2],
                              iw<Y>(4) - c6[3], iw<Y>(5) - c6[4], iw<Y>(6) - c6[5]};
    FaceRef<DIM> R;
    face_ref<DIM, Y>(ld, sk, R);
    Eig<DIM, T> S;
    roe<DIM, T>(ld.after(R.Vf), sk, R, S);
    double cen[NV], del[NV], s6[DIM];  // s6: s_f - central6(s)
#pragma unroll
    for (int v = 0; v < NV; ++v) cen[v] = del[v] = 0.0;
#pragma unroll
    for (int c = 0; c < DIM; ++c) s6[c] = 0.0;
    T mxm = T(0), mx0 = T(0), mxp = T(0);
    double chain = double(S.pI);
    if constexpr (Y == 8) {  // the outermost nodes
        const LD ln = ld.after(chain);
        double V, s0[DIM], s7[DIM];
        ln.metric(0, V, s0);
        ln.metric(7, V, s7);
#pragma unroll
        for (int c = 0; c < DIM; ++c) s6[c] = iw<8>(0) * (s0[c] + s7[c]);
        chain = s6[0];
    }
#pragma unroll
    for (int r = 1; r <= 6; ++r) {
        const LD ln = ld.after(chain);
        Prim<DIM> P;
        double V, s[DIM], U = 0.0;
        ln.prim(r, P);
        ln.metric(r, V, s);
#pragma unroll
        for (int c = 0; c < DIM; ++c) U += P.u[c] * s[c];
        const double w6 = c6[r - 1], wm = w6 * P.rho * U, p = pressure(P, sk.gamma - 1.0), wp = w6 * (p - R.ps);
        cen[0] += wm;
#pragma unroll
        for (int c = 0; c < DIM; ++c) cen[1 + c] = fma(wm, P.u[c], fma(wp, s[c], cen[1 + c]));
        cen[E] = fma(w6 * U, P.E + p, cen[E]);
        const double wV = d5[r - 1] * V;
        del[0] = fma(wV, P.rho - R.Qs[0], del[0]);
#pragma unroll
        for (int c = 0; c < DIM; ++c) del[1 + c] = fma(wV, fma(P.rho, P.u[c], -R.Qs[1 + c]), del[1 + c]);
        del[E] = fma(wV, P.E - R.Qs[E], del[E]);
        if constexpr (Y != 6) {
#pragma unroll
            for (int c = 0; c < DIM; ++c) s6[c] += df[r - 1] * s[c];
        }
        chain = del[0];
        T un, cs;
        node_speeds<DIM, T, LD::CT>(sk, S, P, p, un, cs);
        mxm = fmax(mxm, fabs(un - cs));
        mx0 = fmax(mx0, fabs(un));
        mxp = fmax(mxp, fabs(un + cs));
    }
    if constexpr (Y != 6) {  // F(Q*).(s_f - s6) but for the pressure
        double U = 0.0;
#pragma unroll
        for (int c = 0; c < DIM; ++c) U += R.us[c] * s6[c];
        cen[0] = fma(R.Qs[0], U, cen[0]);
#pragma unroll
        for (int c = 0; c < DIM; ++c) cen[1 + c] = fma(R.Qs[1 + c], U, cen[1 + c]);
        cen[E] = fma(R.Qs[E] + R.ps, U, cen[E]);
    }
#pragma unroll
    for (int c = 0; c < DIM; ++c) cen[1 + c] = fma(R.ps, R.sf[c], cen[1 + c]);
    T w[NV], pa[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) w[v] = T(del[v]);
    project<DIM, T>(S, w, pa);
    const T l0 = fmax(S.sigma * mxm, T(sk.glf[0]));
    const T l1 = fmax(S.sigma * mx0, T(sk.glf[1]));
    const T l2 = fmax(S.sigma * mxp, T(sk.glf[2]));
    pa[0] *= l0;
#pragma unroll
    for (int v = 1; v < E; ++v) pa[v] *= l1;
    pa[E] *= l2;
    T o[NV];
    backproject<DIM, T>(S, pa, o);
#pragma unroll
    for (int v = 0; v < NV; ++v) Fo[v] = fma(double(o[v]), 1.0 / 60.0, cen[v]);
}

template <int DIM, int RECON, int Y, typename T, class LD>
__device__ __forceinline__ void face_flux(const LD& ld, const SchemeK& sk, double (&Fo)[DIM + 2]) {
    if constexpr (RECON == 1)
        face_flux_lu5<DIM, Y, T>(ld, sk, Fo);
    else if constexpr (RECON == 2)
        face_flux_weno7<DIM, Y, T>(ld, sk, Fo);
    else
        face_flux_weno<DIM, Y, T, RECON == 3>(ld, sk, Fo);
}

}  // namespace fpk
