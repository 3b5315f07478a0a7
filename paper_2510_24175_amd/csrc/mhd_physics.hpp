// Device-side pointwise physics of the ideal-MHD finite-volume step.
//
// Conventions (shared with include/mhd.h):
//   primitive  V = (rho, vx, vy, vz, p, Bx, By, Bz, psi)
//   conserved  U = (rho, mx, my, mz, E, Bx, By, Bz, psi)
//   E = p/(gamma-1) + rho|v|^2/2 + |B|^2/2   (magnetic pressure |B|^2/2)
// A face normal to axis d is solved in the cyclic frame (n, t1, t2) =
// (d, d+1, d+2) mod 3.  Everything is templated on the arithmetic type T
// (float or double); reciprocals and square roots go through Num<T>, which
// uses the hardware approximations in FP32, and in FP64 refines the hardware
// estimates.
#pragma once

#include <hip/hip_runtime.h>

namespace mhd {

enum { NQ = 9 };
enum { RHO = 0, VX = 1, VY = 2, VZ = 3, PRS = 4, BX = 5, BY = 6, BZ = 7, PSI = 8 };
enum { MX = 1, MY = 2, MZ = 3, ENG = 4 };
enum { SOLVER_HLL = 0, SOLVER_HLLD = 1 };
// reconstructions: PLM with the minmod or MC limiter, or fifth-order WENO-Z
enum { LIM_MINMOD = 0, LIM_MC = 1, LIM_WENOZ = 2 };

template <typename T> struct Num;

// Type-exact elementary operations (the unsuffixed builtins are the double
// versions and would promote float operands).
template <> struct Num<float> {
    static __device__ __forceinline__ float rcp(float x) { return __builtin_amdgcn_rcpf(x); }
    static __device__ __forceinline__ float sqrt(float x) { return __builtin_amdgcn_sqrtf(x); }
    static __device__ __forceinline__ float rsqrt(float x) { return __builtin_amdgcn_rsqf(x); }
    static __device__ __forceinline__ float abs(float x) { return __builtin_fabsf(x); }
    static __device__ __forceinline__ float min(float a, float b) { return __builtin_fminf(a, b); }
    static __device__ __forceinline__ float max(float a, float b) { return __builtin_fmaxf(a, b); }
    static __device__ __forceinline__ float copysign(float a, float b) { return __builtin_copysignf(a, b); }
    // minmod(a, b) as the median of a, b and 0 (one instruction)
    static __device__ __forceinline__ float minmod(float a, float b) { return __builtin_amdgcn_fmed3f(a, b, 0.0f); }
    static constexpr float eps = 1.1920928955078125e-7f;
    static constexpr float weno_eps = 1e-30f;  // normal, with a finite reciprocal
    static constexpr float big = 3.0e38f;
};

template <> struct Num<double> {
    // reciprocal: the hardware estimate (relative error up to 2^-24.3)
    // refined by two Newton-Raphson steps (e = 1 - x r, r <- r + r e): the IEEE
    // quotient on every one of 2^34 samples of [0.25, 0.5) (the steps commute
    // with powers of two) and of 4M log-uniform ones in [1e-297, 1e297].  A
    // third-order correction of the estimate, one operation shorter, is an ulp
    // off on 186 of them.
    static __device__ __forceinline__ double rcp(double x)
    {
        double r = __builtin_amdgcn_rcp(x);
        double e = __builtin_fma(-x, r, 1.0);
        r = __builtin_fma(r, e, r);
        e = __builtin_fma(-x, r, 1.0);
        return __builtin_fma(r, e, r);
    }
    // square root: one Goldschmidt step from the hardware reciprocal-square-root
    // estimate y ~ 1/sqrt(x) (relative error up to 2^-24.1; g = x y -> sqrt(x),
    // h = y/2 -> 1/(2 sqrt(x)), r = 1/2 - g h, both then within 2^-46) and one
    // residual correction g <- g + (x - g^2) h.  The IEEE root on every one of
    // 2^34 samples of [0.25, 1) (powers of four commute) and of 4M log-uniform
    // ones in [1e-297, 1e297]; with h left at the estimate, one operation
    // shorter, 355 are an ulp off.  x + DBL_MIN keeps the estimate finite at x = 0
    // (result 0); negative x gives NaN; subnormal results lose bits (the
    // kernels' roots are of sums with normal terms).
    static __device__ __forceinline__ double sqrt(double x)
    {
        const double y = __builtin_amdgcn_rsq(x + 2.2250738585072014e-308);
        double g = x * y, h = 0.5 * y;
        const double r = __builtin_fma(-g, h, 0.5);
        g = __builtin_fma(g, r, g);
        h = __builtin_fma(h, r, h);
        return __builtin_fma(__builtin_fma(-g, g, x), h, g);
    }
    // reciprocal square root: y (1 + e/2 + 3/8 e^2), e = 1 - x y^2; within 1.0
    // ulp for normal x > 0 (two Goldschmidt steps: 1.65, three operations
    // more); NaN at 0
    static __device__ __forceinline__ double rsqrt(double x)
    {
        const double y = __builtin_amdgcn_rsq(x);
        const double e = __builtin_fma(-(x * y), y, 1.0);
        return __builtin_fma(y * e, __builtin_fma(e, 0.375, 0.5), y);
    }
    static __device__ __forceinline__ double abs(double x) { return __builtin_fabs(x); }
    static __device__ __forceinline__ double min(double a, double b) { return __builtin_fmin(a, b); }
    static __device__ __forceinline__ double max(double a, double b) { return __builtin_fmax(a, b); }
    static __device__ __forceinline__ double copysign(double a, double b) { return __builtin_copysign(a, b); }
    // minmod(a, b) as the median of a, b and 0 (no FP64 median instruction:
    // four min/max)
    static __device__ __forceinline__ double minmod(double a, double b)
    {
        return __builtin_fmax(__builtin_fmin(a, b), __builtin_fmin(__builtin_fmax(a, b), 0.0));
    }
    static constexpr double eps = 2.220446049250313e-16;
    static constexpr double weno_eps = 1e-40;
    static constexpr double big = 1.0e300;
};

// Selections by sign masks.  A VOP2 v_cndmask_b32, which reads its condition
// from VCC, issues every ~23 cycles in a run of them on gfx950, and a compare
// costs another slow slot; v_bfi_b32 with a mask made by an arithmetic shift of
// a sign bit issues every 4.4 cycles and needs no compare (FP32 add, multiply,
// FMA and 32-bit logic: 2.4; minimum, maximum, median, compare: 4.4; FP64: 4.6;
// FP32 rcp, sqrt, rsq: 8.2; FP64: 16.3; four waves per SIMD, 2.4 GHz).  The
// empty asm hides the mask's origin, or the compiler turns the bit operations
// back into compares and v_cndmask.
template <typename T> struct Bits;

template <> struct Bits<float> {
    static __device__ __forceinline__ unsigned word(float x) { return __builtin_bit_cast(unsigned, x); }
    // all ones where x has its sign bit set, else zero
    static __device__ __forceinline__ unsigned negative(float x) { return opaque((int)word(x) >> 31); }
    // all ones where the sign bits of x and y differ
    static __device__ __forceinline__ unsigned differ(float x, float y) { return opaque((int)(word(x) ^ word(y)) >> 31); }
    // m ? a : b, bit by bit
    static __device__ __forceinline__ float select(unsigned m, float a, float b)
    {
        return __builtin_bit_cast(float, (word(a) & m) | (word(b) & ~m));
    }
    // m ? a : 0
    static __device__ __forceinline__ float keep(unsigned m, float a) { return __builtin_bit_cast(float, word(a) & m); }
    // m ? a : something finite
    static __device__ __forceinline__ float finite_keep(unsigned m, float a) { return keep(m, a); }
    // a with its sign flipped where s is negative
    static __device__ __forceinline__ float flip(float a, float s)
    {
        return __builtin_bit_cast(float, word(a) ^ (word(s) & 0x80000000u));
    }
    static __device__ __forceinline__ unsigned opaque(int m)
    {
        asm("" : "+v"(m));
        return (unsigned)m;
    }
};

template <> struct Bits<double> {
    struct Words { unsigned lo, hi; };
    static __device__ __forceinline__ Words words(double x) { return __builtin_bit_cast(Words, x); }
    static __device__ __forceinline__ unsigned negative(double x) { return Bits<float>::opaque((int)words(x).hi >> 31); }
    static __device__ __forceinline__ unsigned differ(double x, double y)
    {
        return Bits<float>::opaque((int)(words(x).hi ^ words(y).hi) >> 31);
    }
    static __device__ __forceinline__ double select(unsigned m, double a, double b)
    {
        const Words x = words(a), y = words(b);
        return __builtin_bit_cast(double, Words{(x.lo & m) | (y.lo & ~m), (x.hi & m) | (y.hi & ~m)});
    }
    static __device__ __forceinline__ double keep(unsigned m, double a)
    {
        const Words x = words(a);
        return __builtin_bit_cast(double, Words{x.lo & m, x.hi & m});
    }
    static __device__ __forceinline__ double finite_keep(unsigned m, double a)
    {
        const Words x = words(a);
        return __builtin_bit_cast(double, Words{x.lo, x.hi & m});
    }
    static __device__ __forceinline__ double flip(double a, double s)
    {
        const Words x = words(a);
        return __builtin_bit_cast(double, Words{x.lo, x.hi ^ (words(s).hi & 0x80000000u)});
    }
};

// Per-launch constants of the scheme.
template <typename T> struct Phys {
    T gamma;     // adiabatic index
    T gm1;       // gamma - 1
    T inv_gm1;   // 1 / (gamma - 1)
    T inv_gm1m1; // 1 / (gamma - 1) - 1
    T ch;        // GLM wave speed c_h
    T ch2;       // c_h^2
    T half_ich;  // 1 / (2 c_h), 0 when GLM is off
    T half_ch;   // c_h / 2, 0 when GLM is off
    T half_on;   // 1/2, 0 when GLM is off
    unsigned psi_bits; // all ones, 0 when GLM is off
    int glm;     // GLM cleaning on
};

// Conserved -> primitive.  Returns false for rho <= 0, p <= 0 or a
// non-finite value (NaN fails every comparison; infinities fail the upper
// bounds or turn p into NaN or -inf).
template <typename T>
__device__ __forceinline__ bool cons_to_prim(const T *u, const Phys<T> &ph, T *v)
{
    const T rho = u[RHO];
    const T ir = Num<T>::rcp(rho);
    const T vx = u[MX] * ir, vy = u[MY] * ir, vz = u[MZ] * ir;
    const T kin = T(0.5) * (u[MX] * vx + u[MY] * vy + u[MZ] * vz);
    const T mag = T(0.5) * (u[BX] * u[BX] + u[BY] * u[BY] + u[BZ] * u[BZ]);
    const T p = ph.gm1 * (u[ENG] - kin - mag);
    v[RHO] = rho;
    v[VX] = vx;
    v[VY] = vy;
    v[VZ] = vz;
    v[PRS] = p;
    v[BX] = u[BX];
    v[BY] = u[BY];
    v[BZ] = u[BZ];
    v[PSI] = u[PSI];
    const T big = Num<T>::big;
    return (rho > T(0)) & (rho < big) & (p > T(0)) & (p < big) & (Num<T>::abs(u[PSI]) < big);
}

// Limited slope from the backward difference a and the forward difference b:
// minmod(a, b) (zero unless a and b have the same sign, else the one of
// smaller magnitude), or MC = minmod(2a, 2b, (a+b)/2) =
// minmod(2a, minmod(2b, (a+b)/2)).  The limiter is a compile-time parameter
// of the kernels.
template <int LIM, typename T> __device__ __forceinline__ T limited_slope(T a, T b)
{
    if (LIM == LIM_MC) return Num<T>::minmod(T(2) * a, Num<T>::minmod(T(2) * b, T(0.5) * (a + b)));
    return Num<T>::minmod(a, b);
}

// WENO-Z face values of one cell (Borges, Carmona, Costa & Don 2008; p = 1,
// eps = 1e-40 in FP64, 1e-30 in FP32 where 1e-40 is subnormal and its
// reciprocal overflows) from the five cell values v0..v4 centred on it: the
// value at its right face (rgt, x_{i+1/2}) and at its left face (lft,
// x_{i-1/2}).  The three candidate quadratics are fitted to the cell sets
// S0 = {v0,v1,v2}, S1 = {v1,v2,v3}, S2 = {v2,v3,v4}; written around v2 with
// e_k their second differences and G_k half their one-sided first
// differences (G0 = (v0 - 4v1 + 3v2)/2, G1 = (v1 - v3)/2,
// G2 = (3v2 - 4v3 + v4)/2), a candidate's face values are
// v2 + e_k/12 -+ G_k/2 and its Jiang-Shu smoothness indicator is
// beta_k = 13/12 e_k^2 + G_k^2.  Both faces share beta_k and the global
// indicator tau5 = |beta0 - beta2|; their linear weights are mirror images,
// (1, 6, 3)/10 on (S0, S1, S2) for the right face and (3, 6, 1)/10 for the
// left, each scaled by 1 + tau5 / (beta_k + eps).
//
// The weights are multiplied through by (beta0+eps)(beta1+eps)(beta2+eps),
// W_k = prod_{j != k}(beta_j + eps) (beta_k + eps + tau5) (formed as the triple product
// plus tau5 times the pair product), and the linear weights are folded into
// the candidate deviations and the weight sums.  The indicators are formed
// four times as large (one operation fewer); FP64 takes the resulting 64 out
// of the linear weights.  FP64 normalises both faces
// with one reciprocal of the product of the two weight sums: it lies between
// eps^6 and about 4 beta_max^6, so it and its reciprocal stay normal for
// indicators between eps and 1e51 (differences of a few 1e25 between
// neighbouring cell values).  FP32 divides the indicators by a sixteenth of
// their sum and adds 1.6e-17: the largest is then between 5 and 16, products of
// two stay normal, and the floor only binds where an indicator is 1e18 times
// below the sum, that is where its candidate is flat to far below FP32
// resolution of the others'.  The sixteenth keeps the sum's reciprocal normal
// for indicators up to 8e37 (a quarter of FLT_MAX; differences of 5e18 to 9e18);
// larger ones are capped there.  One reciprocal instead of three: 64
// operations and 3 reciprocals a pair instead of 64 and 5 (8.2 cycles each),
// 256^3 stages 1.59 + 1.70 -> 1.50 + 1.60 ms.
template <typename T>
__device__ __forceinline__ void wenoz_pair(T v0, T v1, T v2, T v3, T v4, T &rgt, T &lft)
{
    // e_k, 2 G_k and, below, 4 (beta_k + eps) from the two inner differences (the
    // weights depend on ratios of the indicators only)
    const T da = v2 - v1, db = v2 - v3;
    const T e1 = -(da + db), e0 = (v0 - v1) + da, e2 = (v4 - v3) + db;
    const T G1 = db - da, G0 = e0 + T(2) * da, G2 = e2 + T(2) * db;
    const T c = T(13.0 / 3.0), eps = T(4) * Num<T>::weno_eps;
    // FP64 adds eps first (one fused operation fewer); FP32 last: with eps
    // first the FP32 Brio-Wu tube's error against the oracle moved from 8.8e-6
    // to 1.09e-5 of its 1e-5 bound (other lengths moved either way)
    auto beta = [&](T e, T G) -> T { return sizeof(T) == 8 ? c * e * e + (G * G + eps) : (c * e * e + G * G) + eps; };
    T B0 = beta(e0, G0), B1 = beta(e1, G1), B2 = beta(e2, G2);
    if constexpr (sizeof(T) == 4) {
        // relative to a sixteenth of their sum and at least 1e-18 of the sum,
        // so that the products of two stay normal
        const T top = T(3.4e38), part = T(0.0625), least = T(16) * T(1e-18);
        B0 = Num<T>::min(B0, top);
        B1 = Num<T>::min(B1, top);
        B2 = Num<T>::min(B2, top);
        const T s = Num<T>::rcp(part * B0 + part * B1 + part * B2);
        B0 = B0 * s + least;
        B1 = B1 * s + least;
        B2 = B2 * s + least;
    }
    const T tau = Num<T>::abs(B0 - B2);
    // W_k = B0 B1 B2 + tau5 prod_{j != k} B_j
    const T p12 = B1 * B2, p02 = B0 * B2, p01 = B0 * B1, P = B0 * p12;
    const T w0 = tau * p12 + P, w1 = tau * p02 + P, w2 = tau * p01 + P;
    // candidate deviations from v2 at the two faces, each scaled by its
    // linear weight ((1, 6, 3)/10 right, (3, 6, 1)/10 left), and in FP64 by 1/64
    constexpr T k = sizeof(T) == 8 ? T(0.015625) : T(1);
    const T g0 = T(0.025) * k * G0, g1 = T(0.15) * k * G1, g2 = T(0.025) * k * G2;
    const T d0r = e0 * (T(0.1 / 12.0) * k) + g0, d0l = e0 * (T(0.3 / 12.0) * k) - T(3) * g0;
    const T d1r = e1 * (T(0.05) * k) - g1, d1l = e1 * (T(0.05) * k) + g1;
    const T d2r = e2 * (T(0.3 / 12.0) * k) - T(3) * g2, d2l = e2 * (T(0.1 / 12.0) * k) + g2;
    const T s1 = T(0.6) * k * w1;
    const T nr = w0 * d0r + w1 * d1r + w2 * d2r, nl = w0 * d0l + w1 * d1l + w2 * d2l;
    const T sr = T(0.1) * k * w0 + (T(0.3) * k * w2 + s1), sl = T(0.3) * k * w0 + (T(0.1) * k * w2 + s1);
    if constexpr (sizeof(T) == 8) {
        const T inv = Num<T>::rcp(sr * sl);
        rgt = v2 + nr * (sl * inv);
        lft = v2 + nl * (sr * inv);
    } else {
        rgt = v2 + nr * Num<T>::rcp(sr);
        lft = v2 + nl * Num<T>::rcp(sl);
    }
}

// Fast magnetosonic speed from p, |B|^2, B_n^2 and 1/rho:
// c_f^2 = (a^2 + b^2 + sqrt((a^2 - b^2)^2 + 4 a^2 (b^2 - b_n^2))) / 2.
template <typename T>
__device__ __forceinline__ T fast_speed(T p, T bsq, T bnsq, T gamma, T irho)
{
    const T a2 = gamma * p * irho;
    const T b2 = bsq * irho;
    const T bn2 = bnsq * irho;
    const T dab = a2 - b2;
    T disc = dab * dab + T(4) * a2 * (b2 - bn2);
    disc = Num<T>::max(disc, T(0));
    return Num<T>::sqrt(T(0.5) * (a2 + b2 + Num<T>::sqrt(disc)));
}

// A rotated 8-component state: rho, u (normal), v1, v2, p, bn, b1, b2, with
// its derived energy, total pressure and v.B.
template <typename T> struct RState {
    T rho, u, v1, v2, p, bn, b1, b2;
    T irho, bsq, E, pt, vb;
};

// irho, |B|^2 and total pressure of a rotated state
template <typename T>
__device__ __forceinline__ void rstate_prepare(RState<T> &s)
{
    s.irho = Num<T>::rcp(s.rho);
    s.bsq = s.bn * s.bn + s.b1 * s.b1 + s.b2 * s.b2;
    s.pt = s.p + T(0.5) * s.bsq;
}

// total energy and v.B of a prepared rotated state
template <typename T>
__device__ __forceinline__ void rstate_energy(RState<T> &s, const Phys<T> &ph)
{
    s.E = s.p * ph.inv_gm1 + T(0.5) * s.rho * (s.u * s.u + s.v1 * s.v1 + s.v2 * s.v2) +
          T(0.5) * s.bsq;
    s.vb = s.u * s.bn + s.v1 * s.b1 + s.v2 * s.b2;
}

// physical normal flux (8 comps, slot 5 unused) and conserved vector
template <typename T>
__device__ __forceinline__ void rstate_flux(const RState<T> &s, T *f, T *c)
{
    const T mu = s.rho * s.u;
    f[0] = mu;
    f[1] = mu * s.u + s.pt - s.bn * s.bn;
    f[2] = mu * s.v1 - s.bn * s.b1;
    f[3] = mu * s.v2 - s.bn * s.b2;
    f[4] = (s.E + s.pt) * s.u - s.bn * s.vb;
    f[5] = T(0);
    f[6] = s.u * s.b1 - s.v1 * s.bn;
    f[7] = s.u * s.b2 - s.v2 * s.bn;
    c[0] = s.rho;
    c[1] = mu;
    c[2] = s.rho * s.v1;
    c[3] = s.rho * s.v2;
    c[4] = s.E;
    c[5] = s.bn;
    c[6] = s.b1;
    c[7] = s.b2;
}

template <typename T>
__device__ __forceinline__ T rstate_fast(const RState<T> &s, const Phys<T> &ph)
{
    return fast_speed(s.p, s.bsq, s.bn * s.bn, ph.gamma, s.irho);
}

// HLL flux, Davis bounds clamped to the origin so one formula covers the
// supersonic cases: F = (sR FL - sL FR + sL sR (UR - UL)) / (sR - sL).
// L and R need irho, bsq and pt (rstate_prepare).
template <typename T>
__device__ __forceinline__ void hll_flux(const RState<T> &L, const RState<T> &R,
                                         const Phys<T> &ph, T *F)
{
    RState<T> Le = L, Re = R;
    rstate_energy(Le, ph);
    rstate_energy(Re, ph);
    T FL[8], UL[8], FR[8], UR[8];
    rstate_flux(Le, FL, UL);
    rstate_flux(Re, FR, UR);
    const T cL = rstate_fast(L, ph), cR = rstate_fast(R, ph);
    const T sL = Num<T>::min(Num<T>::min(L.u - cL, R.u - cR), T(0));
    const T sR = Num<T>::max(Num<T>::max(L.u + cL, R.u + cR), T(0));
    const T id = Num<T>::rcp(sR - sL);
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        // slot 5 (B_n) is unused: the interface solve supplies that flux
        if (k == 5) F[k] = T(0);
        else F[k] = (sR * FL[k] - sL * FR[k] + sL * sR * (UR[k] - UL[k])) * id;
    }
}

// One side of an interface in the rotated frame: primitives, transverse field
// squared, total pressure.
template <typename T> struct Side {
    T rho, u, v1, v2, p, b1, b2, bt2, pt;
};

template <typename T> __device__ __forceinline__ void side_prepare(Side<T> &s, T bn)
{
    s.bt2 = s.b1 * s.b1 + s.b2 * s.b2;
    s.pt = s.p + T(0.5) * (bn * bn + s.bt2);
}

// twice the square of the fast speed: with a^2 = g p / rho, b^2 = |B|^2 / rho,
// 2 c_f^2 = a^2 + b^2 + sqrt((a^2 - b^2)^2 + 4 a^2 |B_t|^2 / rho)
template <typename T>
__device__ __forceinline__ T fast_sq2(const Side<T> &s, T bn2, const Phys<T> &ph)
{
    const T ir = Num<T>::rcp(s.rho);
    const T a2 = ph.gamma * s.p * ir, b2 = (bn2 + s.bt2) * ir;
    const T d = a2 - b2;
    const T disc = Num<T>::max(T(4) * a2 * (s.bt2 * ir) + d * d, T(0));
    return (a2 + b2) + Num<T>::sqrt(disc);
}

// total energy density (|B|^2/2 = p_T - p) and v.B
template <typename T>
__device__ __forceinline__ T side_energy(const Side<T> &s, const Phys<T> &ph)
{
    return T(0.5) * s.rho * (s.u * s.u + s.v1 * s.v1 + s.v2 * s.v2) + (s.p * ph.inv_gm1m1 + s.pt);
}
template <typename T> __device__ __forceinline__ T side_vb(const Side<T> &s, T bn)
{
    return s.u * bn + s.v1 * s.b1 + s.v2 * s.b2;
}

// One side of the HLLD single-star state (Miyoshi & Kusano 2005).  With
// m = rho (S - u) and mm = m (S - S_M) > 0, r = 1/sqrt(mm) gives the star
// density's root q = m r (negative on the left; rho* = q^2), 1/q = (S - S_M) r
// and 1/(S - S_M) = q r without further reciprocals.  With w = S_M - u and
// D = mm - B_n^2: v* = v - B_t B_n w / D and B* = B_t (1 + m w / D).
template <typename T> struct Star {
    T v1, v2, b1, b2;
    T sd;    // S - S_M
    T q, r;  // m r, 1/sqrt(m (S - S_M))
    T a;     // (S - u) E - p_T u + B_n v.B, the side's own share of E* (S - S_M)
};

template <typename T>
__device__ __forceinline__ void hlld_star(const Side<T> &s, T S, T su, T m, T w, T sM, T bn, T bn2,
                                          const Phys<T> &ph, Star<T> &o)
{
    o.sd = S - sM;
    const T mm = m * o.sd;
    const T D = mm - bn2;
    // degenerate side, |D| <= 16 eps (mm + B_n^2): 1/D <- 0 keeps its tangential state
    const T tol = T(16) * Num<T>::eps * mm + T(16) * Num<T>::eps * bn2;
    const T x = w * Bits<T>::keep(Bits<T>::negative(tol - Num<T>::abs(D)), Num<T>::rcp(D));
    const T cv = bn * x, cb = m * x;
    o.v1 = s.v1 - s.b1 * cv;
    o.v2 = s.v2 - s.b2 * cv;
    o.b1 = s.b1 + s.b1 * cb;
    o.b2 = s.b2 + s.b2 * cb;
    o.r = Num<T>::rsqrt(mm);
    o.q = m * o.r;
    o.a = su * side_energy(s, ph) - s.pt * s.u + bn * side_vb(s, bn);
}

// HLLD flux (Miyoshi & Kusano 2005; slots rho, m_n, m_1, m_2, E, unused, B_1,
// B_2), outer speeds
// min(u_L, u_R) - max(c_fL, c_fR) and max(u_L, u_R) + max(c_fL, c_fR).  The star
// states satisfy the jump conditions across the outer and the rotational
// waves, so the flux in a star region is the physical flux of the region's
// state, with normal velocity S_M and total pressure p_T*: one state is
// picked and its flux formed, instead of adding the jumps wave by wave.  At
// a supersonic interface (the fan on one side of the face) S_M <- u of the
// upwind side makes that side's star state the side's own state.
template <typename T>
__device__ __forceinline__ void hlld_flux(const Side<T> &L, const Side<T> &R, T bn, const Phys<T> &ph, T *F)
{
    const T bn2 = bn * bn;
    // outer speeds: the slower (faster) normal velocity minus (plus) the
    // larger fast speed (at least as wide as Davis's bounds; keeps the
    // rotational waves inside the fan where Davis's bounds let D cross zero)
    const T cm = Num<T>::sqrt(T(0.5) * Num<T>::max(fast_sq2(L, bn2, ph), fast_sq2(R, bn2, ph)));
    const T sL = Num<T>::min(L.u, R.u) - cm;
    const T sR = Num<T>::max(L.u, R.u) + cm;
    const T suL = sL - L.u, suR = sR - R.u;
    const T mL = suL * L.rho, mR = suR * R.rho;
    // contact speed; the upwind normal velocity when the fan lies on one side
    const T sC = (mR * R.u - mL * L.u + (L.pt - R.pt)) * Num<T>::rcp(mR - mL);
    const T sM = Bits<T>::select(Bits<T>::negative(sR), R.u, Bits<T>::select(Bits<T>::negative(sL), sC, L.u));
    const T wL = sM - L.u, wR = sM - R.u;

    Star<T> sl, sr;
    hlld_star(L, sL, suL, mL, wL, sM, bn, bn2, ph, sl);
    hlld_star(R, sR, suR, mR, wR, sM, bn, bn2, ph, sr);

    // double-star tangential state
    const T iden = Num<T>::rcp(sr.q - sl.q);
    const T wl = -sl.q * iden, wr = sr.q * iden;
    const T si = Bits<T>::flip(iden, bn), sx = -sl.q * sr.q * si;
    const T dv1 = sr.v1 - sl.v1, dv2 = sr.v2 - sl.v2, db1 = sr.b1 - sl.b1, db2 = sr.b2 - sl.b2;
    const T v1ss = sl.v1 + wr * dv1 + si * db1, v2ss = sl.v2 + wr * dv2 + si * db2;
    const T b1ss = sl.b1 + wl * db1 + sx * dv1, b2ss = sl.b2 + wl * db2 + sx * dv2;

    // side of the contact (right where S_M < 0), then the region within it:
    // the rotational wave S_M + |B_n|/q of that side lies across the face
    // when its sign is not S_M's
    const unsigned right = Bits<T>::negative(sM);
    auto pick = [&](T l, T r) -> T { return Bits<T>::select(right, r, l); };
    const T q = pick(sl.q, sr.q), r = pick(sl.r, sr.r), sd = pick(sl.sd, sr.sd), a = pick(sl.a, sr.a);
    const T pts = pick(L.pt + mL * wL, R.pt + mR * wR);
    const T v1s = pick(sl.v1, sr.v1), v2s = pick(sl.v2, sr.v2), b1s = pick(sl.b1, sr.b1), b2s = pick(sl.b2, sr.b2);
    const unsigned dbl = Bits<T>::differ(sM + Num<T>::abs(bn) * (sd * r), sM);
    const T v1 = Bits<T>::select(dbl, v1ss, v1s), v2 = Bits<T>::select(dbl, v2ss, v2s);
    const T b1 = Bits<T>::select(dbl, b1ss, b1s), b2 = Bits<T>::select(dbl, b2ss, b2s);
    const T bs = sM * bn;
    const T vbs = bs + v1s * b1s + v2s * b2s, vb = bs + v1 * b1 + v2 * b2;
    // E* = (a + p_T* S_M - B_n v*.B*) / (S - S_M); E** = E* + q sgn(B_n) (v*.B* - v**.B**)
    const T E = (a + pts * sM - bn * vbs) * (q * r) + Bits<T>::flip(q, bn) * (vbs - vb);
    const T mu = q * q * sM;
    F[0] = mu;
    F[1] = mu * sM + (pts - bn2);
    F[2] = mu * v1 - bn * b1;
    F[3] = mu * v2 - bn * b2;
    F[4] = (E + pts) * sM - bn * vb;
    F[5] = T(0);
    F[6] = sM * b1 - bn * v1;
    F[7] = sM * b2 - bn * v2;
}

// Select a[d] for d in {0,1,2} without indexing a register array (the
// selects fold away when d is a compile-time constant).
template <typename T> __device__ __forceinline__ T pick3(int d, T a0, T a1, T a2)
{
    return d == 0 ? a0 : (d == 1 ? a1 : a2);
}

// Interface flux from two unrotated primitive face states along axis d:
// GLM (B_n, psi) interface solve, MHD solver on the 8 MHD components with
// B_n replaced by B_n*, then F(B_n) = psi*, F(psi) = c_h^2 B_n*.  With
// constrained transport (CT) the normal field is the face's own value bnf
// and F(B_n) = F(psi) = 0.
template <typename T, int SOLVER, bool CT = false>
__device__ __forceinline__ void face_flux(const T *VL, const T *VR, int d, const Phys<T> &ph, T *F,
                                          T bnf = T(0))
{
    // frame (n, t1, t2) = (d, d+1, d+2) mod 3
    const T bnL = pick3(d, VL[BX], VL[BY], VL[BZ]);
    const T bnR = pick3(d, VR[BX], VR[BY], VR[BZ]);
    T bns, psis;
    if (CT) {
        bns = bnf;
        psis = T(0);
    } else {
        // GLM off: half_ich, half_on and half_ch are zero, and the masks keep
        // an infinite or undefined psi (inert, it may have any size) out of
        // their products.  A branch instead spills 12-16 registers of the FP32
        // PLM last stage (512^3 step 8.77 -> 9.31 ms)
        const T dp = Bits<T>::finite_keep(ph.psi_bits, VR[PSI] - VL[PSI]);
        const T sp = Bits<T>::finite_keep(ph.psi_bits, VL[PSI] + VR[PSI]);
        bns = T(0.5) * (bnL + bnR) - dp * ph.half_ich;
        psis = ph.half_on * sp - ph.half_ch * (bnR - bnL);
    }
    // a face state in the frame (RState or Side)
    auto rotate = [&](const T *V, auto &s) {
        s.rho = V[RHO];
        s.u = pick3(d, V[VX], V[VY], V[VZ]);
        s.v1 = pick3(d, V[VY], V[VZ], V[VX]);
        s.v2 = pick3(d, V[VZ], V[VX], V[VY]);
        s.p = V[PRS];
        s.b1 = pick3(d, V[BY], V[BZ], V[BX]);
        s.b2 = pick3(d, V[BZ], V[BX], V[BY]);
    };
    T f[8];
    if constexpr (SOLVER == SOLVER_HLLD) {
        Side<T> L, R;
        rotate(VL, L);
        rotate(VR, R);
        side_prepare(L, bns);
        side_prepare(R, bns);
        hlld_flux(L, R, bns, ph, f);
    } else {
        RState<T> L, R;
        rotate(VL, L);
        rotate(VR, R);
        L.bn = R.bn = bns;
        rstate_prepare(L);
        rstate_prepare(R);
        hll_flux(L, R, ph, f);
    }
    const T fbn = psis;
    F[RHO] = f[0];
    F[ENG] = f[4];
    // unrotate: component x is (n, t2, t1) for d = (0, 1, 2), etc.
    F[MX] = pick3(d, f[1], f[3], f[2]);
    F[MY] = pick3(d, f[2], f[1], f[3]);
    F[MZ] = pick3(d, f[3], f[2], f[1]);
    F[BX] = pick3(d, fbn, f[7], f[6]);
    F[BY] = pick3(d, f[6], fbn, f[7]);
    F[BZ] = pick3(d, f[7], f[6], fbn);
    F[PSI] = CT ? T(0) : ph.ch2 * bns;
}

// Boundary index map of a ghost or interior coordinate m on an axis of n >= 2
// cells: periodic wrap or zero-gradient clamp.  The wrap folds at most twice
// (no integer division), so it is exact for m in [-2n, 3n), which holds every
// position a stencil of an interior cell reaches (m in [-3, n + 3)); other
// coordinates, used only as padding, are clamped into the axis.
__device__ __forceinline__ int remap_index(int m, int n, int periodic)
{
    if (periodic) {
        m = m < 0 ? m + n : m;
        m = m < 0 ? m + n : m;
        m = m >= n ? m - n : m;
        m = m >= n ? m - n : m;
    }
    return m < 0 ? 0 : (m >= n ? n - 1 : m);
}

} // namespace mhd
