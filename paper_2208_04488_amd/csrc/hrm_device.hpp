// hrm_device.hpp -- gfx950 device arithmetic of the hot path: mixture EOS,
// characteristic projection, incremental-stencil WENO, HLLC, HCS
// reconstruction with shock-sensor blending, the positivity-preserving
// interpolation and flux limiters, and the infinite-rate thermal relaxation
// (Wong, Angel & Kiris, arXiv:2208.04488, Sec. 2, Sec. 4, App. C, App. D).
//
// Face arithmetic is templated on R (double, or float for the FP32 variant);
// the node primitives, the flux limiter, every limiter bound check, the
// accumulation and the relaxation are double in both.  Component slots of a
// conservative vector W (Sec. 2): alpha_k rho_k (k < N), rho u_d (d < D), E,
// alpha_k (k < N-1).
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>

namespace hrm {

constexpr int MAXN = 8;

// grid flags (mirror of the public header)
constexpr int F_NO_LIMITERS = 1;
constexpr int F_NO_BLEND = 2;
constexpr int F_FIRST_ORDER = 4;
constexpr int F_FOUR_EQ = 32;  // the four-equation HRM solved directly (first-order HLLC)

// species table with the derived constants every kernel needs
struct EosDev {
    double g[MAXN], cv[MAXN], pinf[MAXN], q[MAXN];
    double ig1[MAXN];   // 1/(gamma_k - 1)
    double gpi1[MAXN];  // gamma_k pinf_k/(gamma_k - 1)
    double cp[MAXN];    // gamma_k c_v,k
};

struct MlpPacked;  // learned interpolation weights (hrm_mlp.hpp)

struct ParDev {
    double eps_weno;
    double eps_i_ar, eps_i_a, hs_i_ar, hs_i_a, hs_i_rc2;
    double eps_f_ar, eps_f_a, eps_f_re, hs_f_ar, hs_f_a, hs_f_re;
    double Cs, qexp, psi;
    double hcs_a, hcs_b, hcs_c;  // eq:reconstructed_G coefficients from psi
    int flags;
    int fast_flux_limiter;    // eps_f >= eps_f^HS for all three quantities
    int fast_interp_limiter;  // eps_i >= eps_i^HS for both quantities
    const MlpPacked* mlp;   // packed network of the learned weights (device), or null
};

// Kernel arguments, read from the kernel-argument segment where they are
// used.  The species table and the parameters (50 to 100 scalar registers
// each) do not fit the 102 scalar registers together: left to itself the
// compiler loads them once and spills them to lanes of vector registers, and
// every use is then a vector instruction (310 v_readlane in a 3D sweep).  The
// empty asm makes the address opaque, so the loads after it (scalar, cached,
// issued beside the vector work) belong to the block of code that uses them
// (256^3 step 14.8 -> 14.2 ms, 1024 x 512 0.306 -> 0.293 ms, the ensemble
// 0.897 -> 0.850 ms).
typedef const __attribute__((address_space(4))) char* KArg;
__device__ __forceinline__ KArg kernel_args() { return (KArg)__builtin_amdgcn_kernarg_segment_ptr(); }
template <typename T>
__device__ __forceinline__ T kload(KArg p)
{
    asm volatile("" : "+s"(p));
    return *(const T*)p;
}

// counters accumulated per thread, flushed once per wave
enum { C_ALG1 = 0, C_ALG2, C_IHS, C_ALG3, C_ALG4, C_FHS, C_RELAX_BAD, C_N };

// The counts of one face (and one cell update) packed into one register, 4
// bits per counter: a face blends at most 2N <= 6 partial densities (Alg. 1)
// and 2 volume-fraction sets (Alg. 2), switches at most twice, limits its
// flux once.  One register instead of seven live through the face.
constexpr unsigned cnt_one(int k) { return 1u << (4 * k); }
__device__ inline unsigned cnt_get(unsigned packed, int k) { return (packed >> (4 * k)) & 15u; }

// A full state: conservative and primitive slots side by side.
template <int N, int D, typename R = double>
struct St {
    R ar[N];   // alpha_k rho_k
    R mom[D];  // rho u_d
    R u[D];
    R p, E;
    double al[N];  // all N volume fractions, al[N-1] = 1 - sum of the others (always double:
                   // a bulk fraction 1 - 1e-8 next to a trace 1e-8 is not representable in float)
    R rho, c, rc2;
};

// a state converted to another arithmetic type
template <int N, int D, typename R, typename S>
__device__ inline St<N, D, R> convert(const St<N, D, S>& s)
{
    St<N, D, R> o;
#pragma unroll
    for (int k = 0; k < N; ++k) {
        o.ar[k] = (R)s.ar[k];
        o.al[k] = s.al[k];
    }
#pragma unroll
    for (int d = 0; d < D; ++d) {
        o.mom[d] = (R)s.mom[d];
        o.u[d] = (R)s.u[d];
    }
    o.p = (R)s.p;
    o.E = (R)s.E;
    o.rho = (R)s.rho;
    o.c = (R)s.c;
    o.rc2 = (R)s.rc2;
    return o;
}

// Sec. 2 mixture EOS: Gam = 1/(gbar-1) = sum alpha_k/(gamma_k-1),
// Pi = gbar pbar/(gbar-1) = sum alpha_k gamma_k pinf_k/(gamma_k-1);
// rho(e - qbar) = Gam p + Pi; rho c^2 = gbar (p + pbar) = p + (p + Pi)/Gam.
template <int N>
__device__ inline void mixture(const EosDev& e, const double* al, double& Gam, double& Pi)
{
    Gam = al[0] * e.ig1[0];
    Pi = al[0] * e.gpi1[0];
#pragma unroll
    for (int k = 1; k < N; ++k) {
        Gam = fma(al[k], e.ig1[k], Gam);
        Pi = fma(al[k], e.gpi1[k], Pi);
    }
}

// 1/x from the hardware reciprocal refined by two Newton steps: within about
// an ulp of the IEEE quotient, in 5 instructions instead of the ~10 of an
// IEEE division.  x must be a normal number (not 0, infinite, NaN or
// subnormal), as the WENO-IS weight sums and the densities and mixture
// Gamma of cells are; elsewhere the IEEE quotient is kept.
__device__ inline double rcp_newton(double x)
{
    double r = __builtin_amdgcn_rcp(x);
    r = fma(fma(-x, r, 1.0), r, r);
    return fma(fma(-x, r, 1.0), r, r);
}

// a/b and sqrt(x) to the bit of the IEEE operations where operands and results
// are normal numbers (and 0 numerators): the reciprocal is refined by one Newton
// step, the root by one of Goldschmidt's coupled iteration, to about 1e-15, and
// the remainder of the quotient (root) that gives, formed with a multiply-add
// (Markstein), corrects the result to 1e-30 before the last rounding.  6 and 11
// instructions instead of the 11 and 18 of the IEEE sequences, whose operand
// scaling for subnormal and huge numbers no state needs.  A zero, infinite or
// NaN divisor gives NaN or infinity; 0 and infinity are their own roots, and a
// negative or NaN radicand gives NaN.  root_rn is the root of a positive number.
__device__ inline double div_rn(double a, double b)
{
    const double r0 = __builtin_amdgcn_rcp(b);
    const double r = fma(fma(-b, r0, 1.0), r0, r0);
    const double q = a * r;
    return fma(fma(-b, q, a), r, q);
}
__device__ inline double root_rn(double x)
{
    const double r = __builtin_amdgcn_rsq(x);
    double g = x * r, h = 0.5 * r;
    const double e = fma(-h, g, 0.5);
    g = fma(g, e, g);
    h = fma(h, e, h);
    return fma(fma(-g, g, x), h, g);
}
__device__ inline double sqrt_rn(double x)
{
    const double r = root_rn(x);
    return __builtin_amdgcn_class(x, 0x260) ? x : r;  // +-0 and +infinity
}
// the quotient in float: the remainder of one that is good to an ulp, times a
// reciprocal rounded once, is off by 3e-15 before the last rounding
// (1024 x 512 in float, two steps 652 -> 642 us, the same bits)
__device__ inline float div_rn(float a, float b)
{
    float r = __builtin_amdgcn_rcpf(b);
    r = fmaf(fmaf(-b, r, 1.0f), r, r);
    const float q = a * r;
    return fmaf(fmaf(-b, q, a), r, q);
}

// x_0^2 + ... + x_{D-1}^2 in one written order; of x_0 and x_1, LAST is the one
// whose square is not rounded
template <int D, typename R, int LAST = 0>
__device__ inline R sum_of_squares(const R* x)
{
#pragma clang fp contract(off)
    if constexpr (D == 1) return x[0] * x[0];
    R s = fma(x[LAST], x[LAST], x[1 - LAST] * x[1 - LAST]);
    if constexpr (D == 3) s = fma(x[2], x[2], s);
    return s;
}

// conservative W[M] -> full state (hot-path step a1).  The multiply-adds are
// written out and no others formed, so that every kernel that takes |u| + c of
// a cell (the separate pass, the sweep that wrote it, the line, the ensemble)
// gets the same bits, and with them the same time step.  The order is kept:
// with rho c^2 off by its last bit 3 to 5 % of an ensemble's time steps were off
// by theirs, which float faces turned into 1e-7 to 1e-5 of the momentum of single
// cells after ten steps.
template <int N, int D>
__device__ inline void state_from_W(const EosDev& e, const double* W, St<N, D>& s)
{
#pragma clang fp contract(off)
    constexpr int IE = N + D, IA = N + D + 1;
    double rho = W[0], rq = W[0] * e.q[0];
    s.ar[0] = W[0];
#pragma unroll
    for (int k = 1; k < N; ++k) {
        s.ar[k] = W[k];
        rho += W[k];
        rq = fma(W[k], e.q[k], rq);
    }
    double asum = 0.0;
#pragma unroll
    for (int k = 0; k < N - 1; ++k) {
        s.al[k] = W[IA + k];
        asum += W[IA + k];
    }
    s.al[N - 1] = 1.0 - asum;
    const double irho = rcp_newton(rho);
    const double m2 = sum_of_squares<D>(W + N);
#pragma unroll
    for (int d = 0; d < D; ++d) {
        s.mom[d] = W[N + d];
        s.u[d] = W[N + d] * irho;
    }
    double Gam, Pi;
    mixture<N>(e, s.al, Gam, Pi);
    const double iG = rcp_newton(Gam);
    s.E = W[IE];
    const double re = fma(-0.5 * m2, irho, W[IE]) - rq;
    s.p = (re - Pi) * iG;
    s.rc2 = fma(fma(re - Pi, iG, Pi), iG, s.p);
    s.rho = rho;
    const double c2 = s.rc2 * irho;
    s.c = c2 == 0.0 ? 0.0 : root_rn(c2);  // a branch: 1 % of the 1000 x 500 step under sqrt_rn's selection
}

// primitive slots (ar, u, p, al[0..N-2]) already set -> the rest of the state;
// POSITIVE: c is asked for only where rho c^2 > 0
template <int N, int D, typename R, int DIR = 0, bool POSITIVE = false>
__device__ inline void complete_from_prim(const EosDev& e, St<N, D, R>& s)
{
#pragma clang fp contract(off)
    R rho = 0, rq = 0;
    double asum = 0.0;
#pragma unroll
    for (int k = 0; k < N; ++k) {
        rho += s.ar[k];
        rq = fma(s.ar[k], (R)e.q[k], rq);
    }
#pragma unroll
    for (int k = 0; k < N - 1; ++k) asum += s.al[k];
    s.al[N - 1] = 1.0 - asum;
    double Gd, Pd;
    mixture<N>(e, s.al, Gd, Pd);
    const R Gam = (R)Gd, Pi = (R)Pd;
    const R u2 = sum_of_squares<D, R, DIR == 1>(s.u);
#pragma unroll
    for (int d = 0; d < D; ++d) s.mom[d] = rho * s.u[d];
    s.rho = rho;
    s.E = fma((R)0.5 * rho, u2, fma(Gam, s.p, Pi)) + rq;
    s.rc2 = s.p + div_rn(s.p + Pi, Gam);
    const R c2 = div_rn(s.rc2, rho);
    s.c = POSITIVE ? root_rn(c2) : sqrt_rn(c2);
}

// rho(e - qbar) of a conservative vector
template <int N, int D>
__device__ inline double rhoe_tilde(const EosDev& e, const double* W)
{
#pragma clang fp contract(off)
    double rho = 0.0, rq = 0.0;
#pragma unroll
    for (int k = 0; k < N; ++k) {
        rho += W[k];
        rq = fma(W[k], e.q[k], rq);
    }
    return W[N + D] - 0.5 * sum_of_squares<D>(W + N) / rho - rq;
}

// num/den for a den as rcp_newton takes it: the hardware reciprocal's
// relative error e (below 5e-8) is divided out as 1 + e + e^2 on the first
// quotient, to within about an ulp of the IEEE one in 5 instructions.
__device__ inline double quot_newton(double num, double den)
{
    const double r = __builtin_amdgcn_rcp(den);
    const double e = fma(-den, r, 1.0);
    const double q = num * r;
    return fma(q, fma(e, e, e), q);
}

// App. C incremental-stencil WENO.  The candidates and the smoothness
// indicators use differences of the stencil only; with d_k the first and e_k
// the second differences, both biased values need five d and four e, and every
// indicator is one square added to the square of an e:
//   4 beta_01 = (13/3) e_i^2 + (d_{i-1/2} + d_{i+1/2})^2, and so on.
// The indicators are scaled by 4 throughout (the weights are unchanged if eps
// is too), eps is the addend the first square is accumulated on, and the
// result is node i plus the weighted deviation of the candidates.  A pair of
// values takes 108 FP64 instructions this way, where the candidates, the
// indicators and the weights each formed from the nodes took 160; the sweeps
// are bound by instruction issue (256^3 step 16.4 -> 14.8 ms, 1024 x 512
// 0.331 -> 0.306 ms, the 4096-problem ensemble 0.938 -> 0.897 ms).
//
// one biased value: u = node i, d1 and d2 the differences across its upwind
// and downwind midpoints (D2 = 2 d2, D6 = 6 d2), e0, e1, e2 the second
// differences about the upwind node, node i and the downwind node, A1 =
// (13/3) e1^2 + eps4 and A2 = (13/3) e2^2 + eps4, B0 = 4 beta_0 + eps4.
// The four weights are scaled by the common product of their denominators
// (and by 32/5), so that one quotient is left; the product spans up to about
// 1e-72..1e58 for the ranges met here, which double holds.
__device__ inline double weno_is_side(double u, double d1, double d2, double D2, double D6, double e0, double e1,
                                      double e2, double A1, double A2, double B0, double eps4)
{
    constexpr double c = 13.0 / 3.0;
    const double D1 = 2.0 * d1, b01 = d1 + d2, b2 = e2 - D2, b3 = e0 + D1;
    const double B1 = fma(D1, D1, eps4), B01 = fma(b01, b01, A1), B2 = fma(b2, b2, A2);
    const double B3 = fma(b3, b3, fma(c * e0, e0, eps4));
    const double t = fma(-2.0, e1, e0 + e2), s = e2 - e0;
    const double tau = fma(s, s, (c * t) * t);
    const double t2 = tau * tau, B23 = B2 * B3, P = (B0 * B1) * B01;
    const double E0 = fma(B0, B01, t2) * (B1 * B23);  // x 3
    const double E1 = fma(B1, B01, t2) * (B0 * B23);  // x 1
    const double E2 = fma(tau, B3, B23) * P;          // x 2
    const double E3 = fma(tau, B2, B23) * P;          // x 2/5
    // four times the candidates' deviations from u, with those factors
    const double F2 = fma(2.0, D2, -e2), F3 = fma(0.6, e0, 0.4 * D1);
    const double num = fma(E0, D6, fma(E1, D1, fma(E2, F2, E3 * F3)));
    const double den = fma(3.0, E0, fma(2.0, E2, fma(0.4, E3, E1)));
    return fma(0.25, quot_newton(num, den), u);
}

// left-biased at i+1/2 from u_{i-2..i+2}
__device__ inline double weno_is(double um2, double um1, double u0, double up1, double up2, double eps)
{
    constexpr double c = 13.0 / 3.0;
    const double d0 = um1 - um2, d1 = u0 - um1, d2 = up1 - u0, d3 = up2 - up1;
    const double e0 = d1 - d0, e1 = d2 - d1, e2 = d3 - d2, eps4 = 4.0 * eps, D2 = 2.0 * d2;
    return weno_is_side(u0, d1, d2, D2, 3.0 * D2, e0, e1, e2, fma(c * e1, e1, eps4), fma(c * e2, e2, eps4),
                        fma(D2, D2, eps4), eps4);
}

// Both biased values at i+1/2 from v[0..5] = u_{i-2..i+3}: the left-biased
// one of v0..v4 and the right-biased one of the mirrored stencil v5..v1,
// whose differences are the same ones with the opposite sign.
__device__ inline void weno_is_pair(const double* v, double eps, double& l, double& r)
{
    constexpr double c = 13.0 / 3.0;
    const double eps4 = 4.0 * eps;
    const double d0 = v[1] - v[0], d1 = v[2] - v[1], d2 = v[3] - v[2], d3 = v[4] - v[3], d4 = v[5] - v[4];
    const double e0 = d1 - d0, e1 = d2 - d1, e2 = d3 - d2, e3 = d4 - d3;
    const double D2 = 2.0 * d2, D6 = 3.0 * D2;
    const double B0 = fma(D2, D2, eps4), A1 = fma(c * e1, e1, eps4), A2 = fma(c * e2, e2, eps4);
    l = weno_is_side(v[2], d1, d2, D2, D6, e0, e1, e2, A1, A2, B0, eps4);
    r = weno_is_side(v[3], -d3, -d2, -D2, -D6, e3, e2, e1, A2, A1, B0, eps4);
}

// FP32 variant: the candidates and smoothness indicators are float and only
// the weighting is done in double, normalised by one reciprocal.
__device__ inline float weno_is_weigh(float s0, float s1, float s2, float s3, float q0, float q1, float q01, float q2,
                                      float q3, float qt, double eps)
{
    const double B0 = (double)q0 + eps, B1 = (double)q1 + eps, B01 = (double)q01 + eps;
    const double B2 = (double)q2 + eps, B3 = (double)q3 + eps, tau = qt;
    const double t2 = tau * tau, B23 = B2 * B3, B0B1 = B0 * B1;
    const double e0 = (15.0 / 32.0) * (B0 * B01 + t2) * B1 * B23;
    const double e1 = (5.0 / 32.0) * (B1 * B01 + t2) * B0 * B23;
    const double e2 = (5.0 / 16.0) * (B2 + tau) * B0B1 * B01 * B3;
    const double e3 = (1.0 / 16.0) * (B3 + tau) * B0B1 * B01 * B2;
    const double inv = rcp_newton(e0 + e1 + e2 + e3);
    return (float)(e0 * inv) * s0 + (float)(e1 * inv) * s1 + (float)(e2 * inv) * s2 + (float)(e3 * inv) * s3;
}

// the FP32 pair shares the candidate (u_i + u_{i+1})/2, beta_0 and the squared
// second differences about i and i+1
__device__ inline void weno_is_pair(const float* v, double eps, float& l, float& r)
{
    using R = float;
    constexpr R c13 = (R)(13.0 / 12.0);
    const R s0 = (R)0.5 * (v[2] + v[3]);
    const R a0 = v[2] - v[3];
    const R q0 = a0 * a0;
    const R dA = v[1] - (R)2 * v[2] + v[3];  // second difference about i
    const R dB = v[2] - (R)2 * v[3] + v[4];  // second difference about i+1
    const R cA = c13 * dA * dA, cB = c13 * dB * dB;
    {
        const R s1 = (R)0.5 * ((R)3 * v[2] - v[1]);
        const R s2 = (R)0.125 * ((R)3 * v[2] + (R)6 * v[3] - v[4]);
        const R s3 = (R)0.125 * ((R)3 * v[0] - (R)10 * v[1] + (R)15 * v[2]);
        const R a1 = v[1] - v[2], b01b = v[1] - v[3], b2b = (R)3 * v[2] - (R)4 * v[3] + v[4];
        const R b3a = v[0] - (R)2 * v[1] + v[2], b3b = v[0] - (R)4 * v[1] + (R)3 * v[2];
        const R t5a = v[4] - (R)4 * v[3] + (R)6 * v[2] - (R)4 * v[1] + v[0];
        const R t5b = v[4] - (R)2 * v[3] + (R)2 * v[1] - v[0];
        const R q1 = a1 * a1;
        const R q01 = cA + (R)0.25 * b01b * b01b;
        const R q2 = cB + (R)0.25 * b2b * b2b;
        const R q3 = c13 * b3a * b3a + (R)0.25 * b3b * b3b;
        const R qt = c13 * t5a * t5a + (R)0.25 * t5b * t5b;
        l = weno_is_weigh(s0, s1, s2, s3, q0, q1, q01, q2, q3, qt, eps);
    }
    {
        const R s1 = (R)0.5 * ((R)3 * v[3] - v[4]);
        const R s2 = (R)0.125 * ((R)3 * v[3] + (R)6 * v[2] - v[1]);
        const R s3 = (R)0.125 * ((R)3 * v[5] - (R)10 * v[4] + (R)15 * v[3]);
        const R a1 = v[4] - v[3], b01b = v[4] - v[2], b2b = (R)3 * v[3] - (R)4 * v[2] + v[1];
        const R b3a = v[5] - (R)2 * v[4] + v[3], b3b = v[5] - (R)4 * v[4] + (R)3 * v[3];
        const R t5a = v[1] - (R)4 * v[2] + (R)6 * v[3] - (R)4 * v[4] + v[5];
        const R t5b = v[1] - (R)2 * v[2] + (R)2 * v[4] - v[5];
        const R q1 = a1 * a1;
        const R q01 = cB + (R)0.25 * b01b * b01b;
        const R q2 = cA + (R)0.25 * b2b * b2b;
        const R q3 = c13 * b3a * b3a + (R)0.25 * b3b * b3b;
        const R qt = c13 * t5a * t5a + (R)0.25 * t5b * t5b;
        r = weno_is_weigh(s0, s1, s2, s3, q0, q1, q01, q2, q3, qt, eps);
    }
}

// wave speed estimates of Sec. 4.1.1 and the contact speed
template <typename R>
__device__ inline R hllc_speeds(R uL, R uR, R pL, R pR, R rhoL, R rhoR, R cL, R cR, R& sL, R& sR)
{
#pragma clang fp contract(off)
    const R ub = (R)0.5 * (uL + uR), cb = (R)0.5 * (cL + cR);
    sL = fmin(ub - cb, uL - cL);
    sR = fmax(ub + cb, uR + cR);
    const R dL = sL - uL, dR = sR - uR;
    return div_rn(fma(-(rhoR * uR), dR, fma(rhoL * uL, dL, pR - pL)), fma(rhoL, dL, -(rhoR * dR)));
}

// Sec. 4.1.1 HLLC for the five-equation model in direction DIR.  Writes
// G = F^HLLC + (0, ..., f_alpha) and returns s_*.
//
// The jumps U*_K - U_K are taken in closed form, with q_K = (s* - u_K) /
// (s_K - s*) = chi_K - 1: q U for the slots that the contact carries, rho s_K
// q for the normal momentum, q (E + p + rho s* (s_K - u_K)) for the energy.
// In double only the side that the flux is taken from is evaluated: K = L for
// s* >= 0, else R (at s* = 0 both sides give the same flux, p* in the normal
// momentum and 0 elsewhere, so either stands for their average).  That needs
// two divisions instead of five and half of the flux arithmetic.
template <int N, int D, int DIR>
__device__ inline double hllc(const St<N, D>& L, const St<N, D>& Rs, double* G)
{
#pragma clang fp contract(off)
    constexpr int IE = N + D, IA = N + D + 1;
    double sL, sR;
    const double ss =
        hllc_speeds<double>(L.u[DIR], Rs.u[DIR], L.p, Rs.p, L.rho, Rs.rho, L.c, Rs.c, sL, sR);
    const bool left = ss >= 0.0;
    auto pick = [&](double a, double b) { return left ? a : b; };
    const double u = pick(L.u[DIR], Rs.u[DIR]), p = pick(L.p, Rs.p), rho = pick(L.rho, Rs.rho);
    const double E = pick(L.E, Rs.E), sk = pick(sL, sR), cap = pick(fmin(0.0, sL), fmax(0.0, sR));
    const double cq = cap * div_rn(ss - u, sk - ss);
#pragma unroll
    for (int k = 0; k < N; ++k) {
        const double a = pick(L.ar[k], Rs.ar[k]);
        G[k] = fma(cq, a, a * u);
    }
    const double m = rho * u;
#pragma unroll
    for (int d = 0; d < D; ++d) {
        const double md = d == DIR ? m : rho * pick(L.u[d], Rs.u[d]);
        G[N + d] = d == DIR ? fma(cq, rho * sk, fma(m, u, p)) : fma(cq, md, md * u);
    }
    const double h = E + p;
    G[IE] = fma(cq, fma(rho * ss, sk - u, h), h * u);
#pragma unroll
    for (int k = 0; k < N - 1; ++k) G[IA + k] = pick(L.al[k], Rs.al[k]) * ss;
    return ss;
}

// The same solver for the faces that keep their order of rounding: the side the
// flux is taken from, or at s* = 0 the mean of both (sign(0) = 0; a flow that is
// symmetric about the face stays so).  In double the jumps are those of the star
// states U*_K = chi_K (...).  In float they are taken in closed form as above:
// chi_K U_K - U_K would round to 0 and drop the star-state correction of the flux
// where |s_K| (a liquid's sound speed) dwarfs |s* - u_K|.  NODES: of two nodes in
// double, where the products u W are rounded.
template <int N, int D, int DIR, typename R, bool NODES = false>
__device__ inline R hllc_kept(const St<N, D, R>& L, const St<N, D, R>& Rs, double* G)
{
#pragma clang fp contract(off)
    constexpr int M = 2 * N + D, IE = N + D, IA = N + D + 1;
    constexpr bool CHI = sizeof(R) == sizeof(double);
    R sL, sR;
    const R uL = L.u[DIR], uR = Rs.u[DIR];
    const R ss = hllc_speeds<R>(uL, uR, L.p, Rs.p, L.rho, Rs.rho, L.c, Rs.c, sL, sR);
    auto from = [&](bool left, double* F) {
#pragma clang fp contract(off)
        auto pick = [&](R a, R b) { return left ? a : b; };
        const R u = pick(uL, uR), p = pick(L.p, Rs.p), rho = pick(L.rho, Rs.rho), E = pick(L.E, Rs.E);
        const R sk = pick(sL, sR), cap = pick(fmin((R)0, sL), fmax((R)0, sR)), d = sk - u;
        const R q = div_rn(CHI ? d : ss - u, sk - ss);  // chi_K, or chi_K - 1
        auto side = [&](R x, R j) {  // u x + cap j
#pragma clang fp contract(off)
            return CHI && NODES ? fma(cap, j, x * u) : fma(x, u, cap * j);
        };
#pragma unroll
        for (int k = 0; k < N; ++k) {
            const R a = pick(L.ar[k], Rs.ar[k]);
            F[k] = side(a, CHI ? fma(q, a, -a) : q * a);
        }
#pragma unroll
        for (int e = 0; e < D; ++e) {
            const R m = pick(L.mom[e], Rs.mom[e]);
            const R f = e == DIR ? fma(m, u, p) : m * u;
            R jump;
            if constexpr (CHI)
                jump = fma(q * rho, e == DIR ? ss : pick(L.u[e], Rs.u[e]), -m);
            else
                jump = e == DIR ? rho * sk * q : q * m;
            F[N + e] = fma(cap, jump, f);
        }
        R jump;
        if constexpr (CHI)
            jump = fma(q, fma(ss - u, fma(rho, ss, div_rn(p, d)), E), -E);
        else
            jump = q * fma(rho * ss, d, E + p);
        F[IE] = side(E + p, jump);
#pragma unroll
        for (int k = 0; k < N - 1; ++k) F[IA + k] = (left ? L.al[k] : Rs.al[k]) * (double)ss;
    };
    from(ss >= (R)0, G);
    if (__builtin_expect(ss == (R)0, 0)) {
        // (at rest under one pressure the two sides are the same)
        bool rest = L.p == Rs.p;
#pragma unroll
        for (int e = 0; e < D; ++e) rest = rest & (L.u[e] == (R)0) & (Rs.u[e] == (R)0);
        if (!rest) {
            double F[M];
            from(false, F);
#pragma unroll
            for (int c = 0; c < M; ++c) G[c] = (R)fma((R)0.5, (R)G[c], (R)0.5 * (R)F[c]);
        }
    }
    return ss;
}

// (1 - t) a + t b in one written order, for values that become a float face's
__device__ inline double blend(double t, double a, double b)
{
#pragma clang fp contract(off)
    return fma(t, b, (1.0 - t) * a);
}

// theta solving (1-theta) a + theta b = min(eps, a) when b < min(eps, a); else 1
__device__ inline double lim_theta(double a, double b, double eps)
{
    const double m = fmin(eps, a);
    return b < m ? (a - m) / (a - b) : 1.0;
}

// rho c^2 of a node read back from its record (which does not hold it: only the
// limiter's rare path asks for it, as a bound of about 1e-9), to an ulp as
// state_from_W forms it
template <int N, int D>
__device__ inline void set_rc2(KArg ke, St<N, D>& s)
{
#pragma clang fp contract(off)
    double Gam, Pi;
    mixture<N>(kload<EosDev>(ke), s.al, Gam, Pi);
    s.rc2 = fma(s.p + Pi, rcp_newton(Gam), s.p);
}

// Completes an interpolated primitive state V and tells whether the limiter
// below would leave it as it is, without looking at the node: every partial
// density and volume fraction at or above eps (then b >= eps >= min(eps, a):
// no blending, and with eps >= eps^HS no hard switch), rho c^2 positive and at
// or above eps^HS, and everything finite (an infinite or NaN slot leaves a
// bound unmet or makes E or rho c^2 infinite or NaN).  Most faces pass; the
// nodes are read from LDS and the limiter runs only where one does not.
template <int N, int D, int DIR, typename R>
__device__ inline bool interp_clean(KArg ke, KArg kp, St<N, D, R>& V)
{
    const EosDev e = kload<EosDev>(ke);
    const ParDev P = kload<ParDev>(kp);
    complete_from_prim<N, D, R, DIR, true>(e, V);
    bool ok = P.fast_interp_limiter != 0;
    ok = ok & (V.rc2 > 0);
#pragma unroll
    for (int k = 0; k < N; ++k) ok = ok & ((double)V.ar[k] >= P.eps_i_ar) & (V.al[k] >= P.eps_i_a);
    return ok & ((double)V.rc2 >= P.hs_i_rc2) & isfinite(V.rc2) & isfinite(V.E);
}

// Sec. 4.3.2 interpolation limiter on an interpolated primitive state V
// (partial densities and volume fractions are blended toward the node state;
// velocity and pressure are kept), then the hard switch to the node state.
// On return V is a complete state (conservative slots, rho, c, rho c^2).
template <int N, int D, int DIR, typename R>
__device__ inline void interp_limit(KArg ke, KArg kp, St<N, D, R>& V, const St<N, D, R>& node, unsigned& cnt)
{
    const EosDev e = kload<EosDev>(ke);
    const ParDev P = kload<ParDev>(kp);
#pragma unroll
    for (int k = 0; k < N; ++k) {  // Alg. 1
        const double a = node.ar[k], b = V.ar[k];
        const double m = fmin(P.eps_i_ar, a);
        if (b < m) {
            const double th = (a - m) / (a - b);
            V.ar[k] = (R)blend(th, a, b);
            cnt += cnt_one(C_ALG1);
        }
    }
    double at[N], asum = 0.0;  // Alg. 2
#pragma unroll
    for (int k = 0; k < N - 1; ++k) {
        at[k] = V.al[k];
        asum += at[k];
    }
    at[N - 1] = 1.0 - asum;
    double th = 1.0;
#pragma unroll
    for (int k = 0; k < N; ++k) th = fmin(th, lim_theta((double)node.al[k], at[k], P.eps_i_a));
    if (th < 1.0) {
#pragma unroll
        for (int k = 0; k < N - 1; ++k) V.al[k] = blend(th, node.al[k], V.al[k]);
        cnt += cnt_one(C_ALG2);
    }
    // hard switch, judged on the completed limited state
    complete_from_prim<N, D, R, DIR>(e, V);
    bool hs = !isfinite(V.rc2) || !isfinite(V.p);
#pragma unroll
    for (int k = 0; k < N; ++k) {
        hs |= !isfinite(V.ar[k]) || !isfinite(V.al[k]);
        hs |= (double)V.ar[k] < fmin(P.hs_i_ar, (double)node.ar[k]);
        hs |= (double)V.al[k] < fmin(P.hs_i_a, (double)node.al[k]);
    }
#pragma unroll
    for (int d = 0; d < D; ++d) hs |= !isfinite(V.u[d]);
    hs |= (double)V.rc2 < fmin(P.hs_i_rc2, (double)node.rc2);
    if (hs) {
#pragma unroll
        for (int k = 0; k < N; ++k) V.ar[k] = node.ar[k];
#pragma unroll
        for (int d = 0; d < D; ++d) V.u[d] = node.u[d];
        V.p = node.p;
#pragma unroll
        for (int k = 0; k < N - 1; ++k) V.al[k] = node.al[k];
        complete_from_prim<N, D, R>(e, V);
        cnt += cnt_one(C_IHS);
    }
}

// all N volume fractions of a conservative vector
template <int N, int D>
__device__ inline void alphas(const double* W, double* al)
{
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < N - 1; ++k) {
        al[k] = W[N + D + 1 + k];
        s += al[k];
    }
    al[N - 1] = 1.0 - s;
}

// Sec. 4.3.2 flux limiter (Alg. 3, Alg. 4, hard switch) at the face between
// nodes L = i and R = i+1.  G pairs are given as the "-" vector (M slots)
// plus the alpha slots of the "+" vector (N-1); the other slots agree.
//   W_i^+     = W_i     - 2 lambda (G^- - F_i)
//   W_{i+1}^- = W_{i+1} + 2 lambda (G^+ - F_{i+1})
// True when the high-order pair's half-cell states (Sec. 4.3.2) are finite
// and at or above every flux-limiter bound: then theta = 1 in Alg. 3 and
// Alg. 4 whatever the first-order states are (b >= eps >= min(eps, a)), the
// hard switch cannot fire (eps >= eps^HS, checked at set-up), and the
// limited pair is the high-order one.  Meaningful only with
// P.fast_flux_limiter.
template <int N, int D, int DIR>
__device__ inline bool flux_limit_clean(KArg ke, KArg kp, const St<N, D>& L, const St<N, D>& R, double lam,
                                        const double* Gho, const double* Gho_p)
{
    constexpr int IE = N + D, IA = N + D + 1;
    const EosDev e = kload<EosDev>(ke);
    const ParDev P = kload<ParDev>(kp);
    if (!P.fast_flux_limiter) return false;
    // the half-cell states W+ (from node i) and W- (from node i+1) are formed
    // slot by slot and checked at once, with running sums for rho, rho q-bar,
    // |rho u|^2 and the volume fractions, instead of being held whole
    const double uL = L.u[DIR], uR = R.u[DIR];
    const double l2 = 2.0 * lam;
    bool ok = true;
    double rp = 0.0, rm = 0.0, qp = 0.0, qm = 0.0;
#pragma unroll
    for (int k = 0; k < N; ++k) {
        const double wp = L.ar[k] - l2 * (Gho[k] - L.ar[k] * uL);
        const double wm = R.ar[k] + l2 * (Gho[k] - R.ar[k] * uR);
        ok = ok & (wp >= P.eps_f_ar) & (wm >= P.eps_f_ar);
        rp += wp;
        rm += wm;
        qp += wp * e.q[k];
        qm += wm * e.q[k];
    }
    double m2p = 0.0, m2m = 0.0;
#pragma unroll
    for (int d = 0; d < D; ++d) {
        const double wp = L.mom[d] - l2 * (Gho[N + d] - (L.mom[d] * uL + (d == DIR ? L.p : 0.0)));
        const double wm = R.mom[d] + l2 * (Gho[N + d] - (R.mom[d] * uR + (d == DIR ? R.p : 0.0)));
        m2p += wp * wp;
        m2m += wm * wm;
    }
    const double Ep = L.E - l2 * (Gho[IE] - (L.E + L.p) * uL);
    const double Em = R.E + l2 * (Gho[IE] - (R.E + R.p) * uR);
    double sp = 0.0, sm = 0.0;
#pragma unroll
    for (int k = 0; k < N - 1; ++k) {
        const double ap = L.al[k] - l2 * Gho[IA + k];
        const double am = R.al[k] + l2 * Gho_p[k];
        ok = ok & (ap >= P.eps_f_a) & (am >= P.eps_f_a);
        sp += ap;
        sm += am;
    }
    ok = ok & (1.0 - sp >= P.eps_f_a) & (1.0 - sm >= P.eps_f_a);
    // rho (e - qbar) >= eps of each half-cell state, times rho: only where that is
    // positive, which a caller's bounds need not say.  An infinite or NaN slot
    // fails its bound or leaves these two products infinite or NaN.
    ok = ok & (rp > 0.0) & (rm > 0.0);
    const double tp = (Ep - qp - P.eps_f_re) * rp - 0.5 * m2p, tm = (Em - qm - P.eps_f_re) * rm - 0.5 * m2m;
    return ok & (tp >= 0.0) & (tm >= 0.0) & isfinite(tp) & isfinite(tm);
}

//
// Every product of the half-cell states is rounded or fused as written here,
// so that all kernels limit a face to the same bits.  FUSED (float faces): the
// high-order states take u W in one rounding with the flux it is subtracted
// from, as the check above does; another last bit of theta there is now and
// then another float in the cells beside the face (1e-5 of their momentum
// after ten steps of a three-species tube).
template <int N, int D, int DIR, bool FUSED>
__device__ inline void flux_limit(KArg ke, KArg kp, const St<N, D>& L, const St<N, D>& R, double lam,
                                  const double* Gho, const double* Gho_p, const double* Glo, const double* Glo_p,
                                  double* G, double* Gp, unsigned& cnt)
{
#pragma clang fp contract(off)
    constexpr int M = 2 * N + D, IE = N + D, IA = N + D + 1;
    const EosDev e = kload<EosDev>(ke);
    const ParDev P = kload<ParDev>(kp);
    double WL[M], WR[M], FL[M], FR[M];
    const double uL = L.u[DIR], uR = R.u[DIR];
#pragma unroll
    for (int k = 0; k < N; ++k) {
        WL[k] = L.ar[k];
        WR[k] = R.ar[k];
        FL[k] = L.ar[k] * uL;
        FR[k] = R.ar[k] * uR;
    }
#pragma unroll
    for (int d = 0; d < D; ++d) {
        WL[N + d] = L.mom[d];
        WR[N + d] = R.mom[d];
        FL[N + d] = d == DIR ? fma(L.mom[d], uL, L.p) : L.mom[d] * uL;
        FR[N + d] = d == DIR ? fma(R.mom[d], uR, R.p) : R.mom[d] * uR;
    }
    WL[IE] = L.E;
    WR[IE] = R.E;
    FL[IE] = (L.E + L.p) * uL;
    FR[IE] = (R.E + R.p) * uR;
#pragma unroll
    for (int k = 0; k < N - 1; ++k) {
        WL[IA + k] = L.al[k];
        WR[IA + k] = R.al[k];
        FL[IA + k] = 0.0;
        FR[IA + k] = 0.0;
    }
    const double l2 = 2.0 * lam;
    // half-cell states of the first-order pair (reference values)
    double Wp_lo[M], Wm_lo[M];
#pragma unroll
    for (int c = 0; c < M; ++c) {
        const double gp = c >= IA ? Glo_p[c - IA] : Glo[c];
        Wp_lo[c] = fma(-l2, Glo[c] - FL[c], WL[c]);
        Wm_lo[c] = fma(l2, gp - FR[c], WR[c]);
    }
    double ap_lo[N], am_lo[N];
    alphas<N, D>(Wp_lo, ap_lo);
    alphas<N, D>(Wm_lo, am_lo);
    const double rep_lo = rhoe_tilde<N, D>(e, Wp_lo), rem_lo = rhoe_tilde<N, D>(e, Wm_lo);

    // Alg. 3
    double Wp[M], Wm[M];
#pragma unroll
    for (int c = 0; c < M; ++c) {
        const double gp = c >= IA ? Gho_p[c - IA] : Gho[c];
        double jp = Gho[c] - FL[c], jm = gp - FR[c];
        if constexpr (FUSED)
            if (c < N || c == IE) {
                jp = fma(-uL, c < N ? L.ar[c < N ? c : 0] : L.E + L.p, Gho[c]);
                jm = fma(-uR, c < N ? R.ar[c < N ? c : 0] : R.E + R.p, Gho[c]);
            }
        Wp[c] = fma(-l2, jp, WL[c]);
        Wm[c] = fma(l2, jm, WR[c]);
    }
    double th = 1.0;
#pragma unroll
    for (int k = 0; k < N; ++k) {
        th = fmin(th, lim_theta(Wp_lo[k], Wp[k], P.eps_f_ar));
        th = fmin(th, lim_theta(Wm_lo[k], Wm[k], P.eps_f_ar));
    }
    {
        double ap[N], am[N];
        alphas<N, D>(Wp, ap);
        alphas<N, D>(Wm, am);
#pragma unroll
        for (int k = 0; k < N; ++k) {
            th = fmin(th, lim_theta(ap_lo[k], ap[k], P.eps_f_a));
            th = fmin(th, lim_theta(am_lo[k], am[k], P.eps_f_a));
        }
    }
    if (th < 1.0) cnt += cnt_one(C_ALG3);
    // When Alg. 3 leaves theta = 1, G* = G^ho and W* = W^ho exactly.  If Alg. 4
    // also gives 1 and everything is finite, the hard switch cannot fire
    // (eps >= eps^HS, checked at context creation), so G** = G^ho: return
    // without rebuilding the half-cell states twice more.
    if (P.fast_flux_limiter && th == 1.0) {
        const double rep = rhoe_tilde<N, D>(e, Wp), rem = rhoe_tilde<N, D>(e, Wm);
        const double t2 = fmin(lim_theta(rep_lo, rep, P.eps_f_re), lim_theta(rem_lo, rem, P.eps_f_re));
        bool fin = isfinite(rep) && isfinite(rem) && isfinite(rep_lo) && isfinite(rem_lo);
#pragma unroll
        for (int c = 0; c < M; ++c) fin = fin && isfinite(Gho[c]) && isfinite(Wp_lo[c]) && isfinite(Wm_lo[c]);
#pragma unroll
        for (int k = 0; k < N - 1; ++k) fin = fin && isfinite(Gho_p[k]);
        if (t2 == 1.0 && fin) {
#pragma unroll
            for (int c = 0; c < M; ++c) G[c] = Gho[c];
#pragma unroll
            for (int k = 0; k < N - 1; ++k) Gp[k] = Gho_p[k];
            return;
        }
    }
    double Gs[M], Gsp[N > 1 ? N - 1 : 1];
#pragma unroll
    for (int c = 0; c < M; ++c) Gs[c] = blend(th, Glo[c], Gho[c]);
#pragma unroll
    for (int k = 0; k < N - 1; ++k) Gsp[k] = blend(th, Glo_p[k], Gho_p[k]);

    // Alg. 4
#pragma unroll
    for (int c = 0; c < M; ++c) {
        const double gp = c >= IA ? Gsp[c - IA] : Gs[c];
        Wp[c] = fma(-l2, Gs[c] - FL[c], WL[c]);
        Wm[c] = fma(l2, gp - FR[c], WR[c]);
    }
    const double th2 = fmin(lim_theta(rep_lo, rhoe_tilde<N, D>(e, Wp), P.eps_f_re),
                            lim_theta(rem_lo, rhoe_tilde<N, D>(e, Wm), P.eps_f_re));
    if (th2 < 1.0) cnt += cnt_one(C_ALG4);
#pragma unroll
    for (int c = 0; c < M; ++c) G[c] = blend(th2, Glo[c], Gs[c]);
#pragma unroll
    for (int k = 0; k < N - 1; ++k) Gp[k] = blend(th2, Glo_p[k], Gsp[k]);

    // hard switch on the final half-cell states
#pragma unroll
    for (int c = 0; c < M; ++c) {
        const double gp = c >= IA ? Gp[c - IA] : G[c];
        Wp[c] = fma(-l2, G[c] - FL[c], WL[c]);
        Wm[c] = fma(l2, gp - FR[c], WR[c]);
    }
    bool hs = false;
#pragma unroll
    for (int c = 0; c < M; ++c) hs |= !isfinite(G[c]);
#pragma unroll
    for (int k = 0; k < N - 1; ++k) hs |= !isfinite(Gp[k]);
    double ap[N], am[N];
    alphas<N, D>(Wp, ap);
    alphas<N, D>(Wm, am);
#pragma unroll
    for (int k = 0; k < N; ++k) {
        hs |= Wp[k] < fmin(P.hs_f_ar, Wp_lo[k]);
        hs |= Wm[k] < fmin(P.hs_f_ar, Wm_lo[k]);
        hs |= ap[k] < fmin(P.hs_f_a, ap_lo[k]);
        hs |= am[k] < fmin(P.hs_f_a, am_lo[k]);
    }
    const double rep = rhoe_tilde<N, D>(e, Wp), rem = rhoe_tilde<N, D>(e, Wm);
    hs |= !isfinite(rep) || !isfinite(rem);
    hs |= rep < fmin(P.hs_f_re, rep_lo);
    hs |= rem < fmin(P.hs_f_re, rem_lo);
    if (hs) {
        cnt += cnt_one(C_FHS);
#pragma unroll
        for (int c = 0; c < M; ++c) G[c] = Glo[c];
#pragma unroll
        for (int k = 0; k < N - 1; ++k) Gp[k] = Glo_p[k];
    }
}

constexpr int BC_PERIODIC = 1, BC_DIRICHLET = 2;

// ghost index map: transmissive copies the edge cell, periodic wraps
// (Dirichlet ghosts are read from the boundary-state array instead)
__device__ inline int map_bc(int g, int n, int lo, int hi)
{
    if (g < 0) return lo == 1 ? ((g % n) + n) % n : 0;
    if (g >= n) return hi == 1 ? g % n : n - 1;
    return g;
}

// the packed counts of a thread (cnt_one), summed over the wave as below
__device__ inline void flush_counters(unsigned packed, unsigned long long* dst);

// sum each counter over the wave, one atomic per non-zero counter.  Most
// counters are zero on every lane of most waves: a ballot skips those (the
// branch is wave-uniform), and the others are summed in 32 bits (a lane's
// counts stay far below 2^26 per launch) by lane permutes.
__device__ inline void flush_counters(const unsigned* c, unsigned long long* dst)
{
    const int lane = __lane_id();
#pragma unroll
    for (int k = 0; k < C_N; ++k) {
        if (__ballot(c[k] != 0u) == 0ull) continue;
        int v = (int)c[k];
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) v += __builtin_amdgcn_ds_bpermute((lane ^ off) << 2, v);
        if (lane == 0) atomicAdd(&dst[k], (unsigned long long)(unsigned)v);
    }
}

__device__ inline void flush_counters(unsigned packed, unsigned long long* dst)
{
    if (__ballot(packed != 0u) == 0ull) return;
    unsigned c[C_N];
#pragma unroll
    for (int k = 0; k < C_N; ++k) c[k] = cnt_get(packed, k);
    flush_counters(c, dst);
}

// NaN-propagating max (a NaN anywhere makes the result NaN)
__device__ inline double nmax(double a, double b) { return a != a ? a : (b != b ? b : fmax(a, b)); }

// block-wide max of D values over the bs threads of the workgroup (a multiple of
// 64); the result is valid in thread 0; sh holds >= bs / 64 * D doubles
template <int D>
__device__ inline void block_max(double* m, double* sh, int bs = (int)blockDim.x)
{
#pragma unroll
    for (int d = 0; d < D; ++d)
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) m[d] = nmax(m[d], __shfl_xor(m[d], off, 64));
    const int w = threadIdx.x >> 6;
    if (__lane_id() == 0)
#pragma unroll
        for (int d = 0; d < D; ++d) sh[w * D + d] = m[d];
    __syncthreads();
    if (threadIdx.x == 0)
        for (int i = 1; i < bs >> 6; ++i)
#pragma unroll
            for (int d = 0; d < D; ++d) m[d] = nmax(m[d], sh[i * D + d]);
}

// Sec. 4.2 infinite-rate thermal relaxation of one cell (species 0 is the
// only stiffened gas): A p^2 + B p + C = 0 (eq:Ap_Bp_Cp_1..3), positive root
// (taken as 2C/(-B - sqrt) when B > 0), T from eq:T_relax_e.  relaxed_pT
// returns p* and T* from W[0 .. N+D] (false when rho(e - qbar) <= 0 or no
// positive root exists); relax_cell then sets alpha_k = alpha_k rho_k /
// rho_k(p, T) for k < N-1, and leaves W unchanged where relaxed_pT fails.
// The root is ill-conditioned in a liquid at low pressure (its condition number
// grows like gamma_1 pinf_1 / p), so this function evaluates each formula in
// the order written, with divisions and roots that round as the IEEE ones
// do (div_rn, sqrt_rn) and no FMA contraction: its rounding is then
// reproducible by any plain double-precision evaluation of the same formulas.
template <int N, int D>
__device__ inline bool relaxed_pT(const EosDev& e, const double* W, double& p_out, double& T_out)
{
#pragma clang fp contract(off)
    constexpr int IE = N + D;
    double rho = 0.0;
#pragma unroll
    for (int k = 0; k < N; ++k) rho += W[k];
    double cvb = 0.0, cpb = 0.0, qb = 0.0, Y0 = 0.0;
#pragma unroll
    for (int k = 0; k < N; ++k) {
        const double Y = div_rn(W[k], rho);  // mass fraction
        cvb += Y * e.cv[k];
        cpb += Y * e.g[k] * e.cv[k];
        qb += Y * e.q[k];
        if (k == 0) Y0 = Y;
    }
    double m2 = 0.0;
#pragma unroll
    for (int d = 0; d < D; ++d) m2 += W[N + d] * W[N + d];
    const double re = W[IE] - div_rn(0.5 * m2, rho) - rho * qb;  // rho (e - qbar)
    if (!(re > 0.0) || !(rho > 0.0)) return false;
    const double p1 = e.pinf[0];
    const double R1 = e.g[0] * e.cv[0] - e.cv[0];  // c_p1 - c_v1
    const double A = cvb;
    const double B = -(re * (cpb - cvb) - p1 * cvb - p1 * Y0 * R1);
    const double C = -re * p1 * ((cpb - cvb) - Y0 * R1);
    const double disc = B * B - 4.0 * A * C;
    double p;
    if (B <= 0.0)
        p = div_rn(-B + sqrt_rn(disc), 2.0 * A);
    else
        p = div_rn(2.0 * C, -B - sqrt_rn(disc));
    if (!(p > 0.0) || !isfinite(p)) return false;
    const double e_t = div_rn(re, rho);
    const double T = div_rn(e_t, div_rn(Y0 * (p + e.g[0] * p1) * e.cv[0], p + p1) + cvb - Y0 * e.cv[0]);
    if (!(T > 0.0) || !isfinite(T)) return false;
    p_out = p;
    T_out = T;
    return true;
}

template <int N, int D>
__device__ inline bool relax_cell(const EosDev& e, double* W)
{
#pragma clang fp contract(off)
    constexpr int IA = N + D + 1;
    double p, T;
    if (!relaxed_pT<N, D>(e, W, p, T)) return false;
#pragma unroll
    for (int k = 0; k < N - 1; ++k) {
        const double rk = div_rn(p + e.pinf[k], (e.g[k] - 1.0) * e.cv[k] * T);  // rho_k(p, T)
        W[IA + k] = div_rn(W[k], rk);
    }
    return true;
}

// Sec. 3: pressure and sound speed of the four-equation HRM from
// alpha_k rho_k, rho u and E.  p is the relaxed p* (eq:p_relax).  c^2 of
// eq:4_eqn_sos takes Psi_k and Gamma from the implicit derivative of the
// relaxation quadratic; scaled by rho it reads F(p) = S_v p^2 + B' p + C' with
//   S_v = sum m_k c_vk,  S_R = sum m_k (c_pk - c_vk),  S_2 = S_R - m_1 (c_p1 - c_v1),
//   B' = -(re S_R - pinf_1 S_v - pinf_1 m_1 (c_p1 - c_v1)),  C' = -re pinf_1 S_2,
// re = rho (e - qbar) = sum m_k (e - q_k) and m_k = alpha_k rho_k.  Summing
// Y_k dF/dm_k and using F(p) = 0 gives sum Y_k Psi_k = (re/rho) X and
// Gamma = X with X = (S_R p + pinf_1 S_2) / F'(p); and F'(p) = 2 S_v p + B' =
// S_v p - C'/p.  So
//   c^2 = p (re + p) (S_R p + pinf_1 S_2) / (rho (S_v p^2 + re pinf_1 S_2)),
// a quotient of positive terms (no cancellation, unlike 2 A_p p + B_p).
// p = c = NaN outside the admissible set.  Written out as state_from_W is: the
// time step is taken from this c, in the pass before the first step and in the
// kernels that take one, and has to be the same.
template <int N, int D>
__device__ inline double hrm4_c(const EosDev& e, const St<N, D>& s, double p)
{
#pragma clang fp contract(off)
    double rho = 0.0, Sv = 0.0, SR = 0.0, rq = 0.0;
#pragma unroll
    for (int k = 0; k < N; ++k) {
        rho += s.ar[k];
        Sv = fma(s.ar[k], e.cv[k], Sv);
        SR = fma(s.ar[k], e.cp[k] - e.cv[k], SR);
        rq = fma(s.ar[k], e.q[k], rq);
    }
    const double re = s.E - div_rn(0.5 * sum_of_squares<D>(s.mom), rho) - rq;
    const double S2 = fma(-s.ar[0], e.cp[0] - e.cv[0], SR);
    const double p1 = e.pinf[0];
    return sqrt_rn(div_rn(p * (re + p) * fma(p1, S2, SR * p), rho * fma(re * p1, S2, Sv * p * p)));
}

template <int N, int D>
__device__ inline void hrm4_pc(const EosDev& e, const St<N, D>& s, double& p, double& c)
{
    double w[N + D + 1], T;
#pragma unroll
    for (int k = 0; k < N; ++k) w[k] = s.ar[k];
#pragma unroll
    for (int d = 0; d < D; ++d) w[N + d] = s.mom[d];
    w[N + D] = s.E;
    if (relaxed_pT<N, D>(e, w, p, T))
        c = hrm4_c<N, D>(e, s, p);
    else
        p = c = __builtin_nan("");
}

// A cell's slot of -(G_{i+1/2} - G_{i-1/2}) / dx, the sum of two directions' and
// its Shu-Osher stage a W^n + b (W^s + dt L): one written order in every kernel
// that takes a step.  (An addition that may be contracted takes a product from a
// function that may not: the sum needs its own.)
__device__ inline double flux_difference(double gr, double gl, double idx)
{
#pragma clang fp contract(off)
    return -(gr - gl) * idx;
}
__device__ inline double add_direction(double L, double next)
{
#pragma clang fp contract(off)
    return L + next;
}
__device__ inline double stage_value(double a, double b, double wn, double ws, double dt, double L)
{
    return fma(a, wn, b * fma(dt, L, ws));
}

struct DtArgs {
    int D;
    double dx[3];
    double cfl, dt_fixed, t_end;
};

// Sec. 4.1.2: tau_d = maxs_d / dx_d, dt = CFL / sum tau (or the fixed step),
// lambda_d = dt / (sigma_d dx_d); clipped to t_end with the device time slot[4]
__device__ inline void dt_from_max(const double* maxs, const DtArgs& a, double* slot)
{
    double tau[3] = {0.0, 0.0, 0.0}, ts = 0.0;
    for (int d = 0; d < a.D; ++d) {
        tau[d] = maxs[d] / a.dx[d];
        ts += tau[d];
    }
    double dt = a.dt_fixed > 0.0 ? a.dt_fixed : a.cfl / ts;
    const double t = slot[4];
    if (a.t_end > 0.0 && t + dt > a.t_end) dt = fmax(a.t_end - t, 0.0);
    slot[0] = dt;
    for (int d = 0; d < 3; ++d) slot[1 + d] = d < a.D ? dt / ((tau[d] / ts) * a.dx[d]) : 0.0;
    slot[4] = a.t_end > 0.0 && t + dt >= a.t_end ? a.t_end : t + dt;
}

}  // namespace hrm
