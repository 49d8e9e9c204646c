// hrm_face.hpp -- one midpoint i+1/2 of the PP-WCNS-IS hyperbolic operator
// (arXiv:2208.04488 Sec. 4.1.1, Sec. 4.3, App. C, App. D), evaluated by one
// thread from the primitive data of the six nodes i-2..i+3 staged in LDS.
#pragma once

#include "hrm_device.hpp"
#include "hrm_mlp.hpp"

namespace hrm {

// LDS node record: the conservative vector W (M slots), then u_d (D),
// p, rho, c (p and c those of the four-equation HRM where that is solved: once
// per node here, not once per face and side).  rho c^2, which only the rare
// path of the limiter asks for, is formed there: one field less lets the 3D y-
// and z-sweeps' 16 x 16 tiles fit four workgroups per CU.
template <int N, int D>
struct NodeFields {
    static constexpr int M = 2 * N + D;
    static constexpr int U = M, P = M + D, RHO = P + 1, C = P + 2;
    static constexpr int COUNT = C + 1;
};

// node j of the stencil, field f; NS = LDS stride between consecutive nodes,
// FS = stride between fields
template <int NS, int FS>
__device__ inline double nodev(const double* nd, int j, int f)
{
    return nd[j * NS + f * FS];
}

template <int N, int D, int NS, int FS>
__device__ inline void load_node(const double* nd, int j, St<N, D>& s)
{
    using F = NodeFields<N, D>;
    constexpr int IE = N + D, IA = N + D + 1;
    double asum = 0.0;
#pragma unroll
    for (int k = 0; k < N; ++k) s.ar[k] = nodev<NS, FS>(nd, j, k);
#pragma unroll
    for (int d = 0; d < D; ++d) {
        s.mom[d] = nodev<NS, FS>(nd, j, N + d);
        s.u[d] = nodev<NS, FS>(nd, j, F::U + d);
    }
    s.E = nodev<NS, FS>(nd, j, IE);
#pragma unroll
    for (int k = 0; k < N - 1; ++k) {
        s.al[k] = nodev<NS, FS>(nd, j, IA + k);
        asum += s.al[k];
    }
    s.al[N - 1] = 1.0 - asum;
    s.p = nodev<NS, FS>(nd, j, F::P);
    s.rho = nodev<NS, FS>(nd, j, F::RHO);
    s.c = nodev<NS, FS>(nd, j, F::C);
}

// the pair of interpolated values at i+1/2 from v[0..5] = nodes i-2..i+3:
// App. C weights (WT = 0), or the learned weights (WT = 1) with App. C as the
// fallback where a learned weight is not finite.  WT = 1 must be reached by
// every lane of the wave (matrix-core evaluation).
template <typename R, int WT>
__device__ inline void interp_pair(const R* v, double eps, const MlpPacked* mlp, R& l, R& r)
{
    if constexpr (WT == 0) {
        weno_is_pair(v, eps, l, r);
    } else {
        const R ul[5] = {v[0], v[1], v[2], v[3], v[4]};
        const R ur[5] = {v[5], v[4], v[3], v[2], v[1]};
        float xl[5], xr[5], zl[3], zr[3], wl[3], wr[3];
        // one side after the other: with both networks' inputs and logits live at
        // once the sweeps of two species keep 21 registers in scratch (1024 x 512,
        // two steps: 946 -> 864 us)
        mlp_inputs(ul, xl);
        mlp_logits(mlp, xl, zl);
        l = mlp_omega(zl, xl, wl) ? mlp_value(ul, wl) : weno_is(v[0], v[1], v[2], v[3], v[4], eps);
        mlp_inputs(ur, xr);
        mlp_logits(mlp, xr, zr);
        r = mlp_omega(zr, xr, wr) ? mlp_value(ur, wr) : weno_is(v[5], v[4], v[3], v[2], v[1], eps);
    }
}

// numerator and denominator (both >= 0) of the shock sensor's normalised
// fourth-order second derivative (Sec. 4.3.1)
__device__ inline void sensor_parts(double v0, double v1, double v2, double v3, double v4, double& num, double& den)
{
    const double a = v1 + v3, y = fma(30.0, v2, v0 + v4);
    num = fabs(fma(16.0, a, -y));
    den = fabs(fma(16.0, a, y));
}

// the ratio itself; a zero denominator (a liquid under tension) gives 1 if
// the numerator is non-zero, else 0
__device__ inline double sensor_ratio(double num, double den)
{
    return den > 0.0 ? num / den : (num > 0.0 ? 1.0 : 0.0);
}

// product of the mean ratios of density and pressure over the two nodes of
// the face: one quotient for the four ratios, unless the product of their
// denominators leaves the range where it is a normal number
__device__ inline double sensor_product(const double* r, const double* p)
{
    double n[4], d[4];
    sensor_parts(r[0], r[1], r[2], r[3], r[4], n[0], d[0]);
    sensor_parts(r[1], r[2], r[3], r[4], r[5], n[1], d[1]);
    sensor_parts(p[0], p[1], p[2], p[3], p[4], n[2], d[2]);
    sensor_parts(p[1], p[2], p[3], p[4], p[5], n[3], d[3]);
    const double dr = d[0] * d[1], dp = d[2] * d[3], dd = dr * dp;
    if (__builtin_expect(dr > 1e-140 && dp > 1e-140 && dd < 1e290, 1))
        return 0.25 * quot_newton(fma(n[0], d[1], n[1] * d[0]) * fma(n[2], d[3], n[3] * d[2]), dd);
    return 0.25 * (sensor_ratio(n[0], d[0]) + sensor_ratio(n[1], d[1])) *
           (sensor_ratio(n[2], d[2]) + sensor_ratio(n[3], d[3]));
}

// The same product ratio by ratio, for float faces and learned weights.  The
// blending weight that comes of it is rounded to float and multiplies fluxes of
// the size of a liquid's pressure, so another last bit here is now and then
// another float there: 1e-5 of the momentum of single cells (three species, ten
// steps).  Hence one written order, whose products are fused as written.
__device__ inline double sensor_ratio_kept(double v0, double v1, double v2, double v3, double v4)
{
    const double num = fabs(fma(16.0, v3, fma(-30.0, v2, fma(16.0, v1, -v0))) - v4);
    const double den = fabs(fma(16.0, v3, fma(30.0, v2, fma(16.0, v1, v0))) + v4);
    return den > 1e-290 ? num * rcp_newton(den) : sensor_ratio(num, den);
}
__device__ inline double sensor_product_kept(const double* r, const double* p)
{
#pragma clang fp contract(off)
    const double sr = 0.5 * (sensor_ratio_kept(r[1], r[2], r[3], r[4], r[5]) +
                             sensor_ratio_kept(r[0], r[1], r[2], r[3], r[4]));
    const double sp = 0.5 * (sensor_ratio_kept(p[1], p[2], p[3], p[4], p[5]) +
                             sensor_ratio_kept(p[0], p[1], p[2], p[3], p[4]));
    return sr * sp;
}

// HCS reconstruction (eq:reconstructed_G) of a slot from its midpoint value t and
// the sums of the node pairs (i, i+1), (i-1, i+2) and (i-2, i+3), blended with t
// by sig; one written order, as above
template <typename R>
__device__ inline R hcs_blend(const ParDev& P, R sig, R t, R g23, R g14, R g05)
{
#pragma clang fp contract(off)
    const R h = fma(-(R)P.hcs_c, g05, fma((R)P.hcs_b, g14, fma((R)P.psi, t, -((R)P.hcs_a * g23))));
    return fma(sig, t, ((R)1 - sig) * h);
}

// Output: G = G^{**,-}_{i+1/2} (M slots) and Gp = alpha slots of G^{**,+}.
// ke and kp: the species table and the parameters in the kernel arguments.
// R is the face arithmetic type; node data, the flux limiter and the outputs
// are double.  LOW = 0 leaves out the first-order and direct-HRM branches
// (selected by flags) for callers that never take them, LOW = 2 leaves out
// everything else for callers that only take those.  Always inlined:
// a call would spill the whole face state around it.
template <int N, int D, int DIR, int NS, int FS, typename R, int WT = 0, int LOW = 1>
__device__ __forceinline__ void face_flux(const double* nd, KArg ke, KArg kp, double lam, double* G, double* Gp,
                                          unsigned& cnt)
{
    static_assert(2 * N <= 15, "per-face counts are packed 4 bits per counter");
    using F = NodeFields<N, D>;
    constexpr int M = 2 * N + D, IE = N + D, IA = N + D + 1;
    constexpr int NA = N > 1 ? N - 1 : 1;
    // FP32: the characteristic fields are interpolated as deviations from
    // node i, formed in double.  WENO-IS is translation-equivariant (the
    // smoothness indicators use differences only and the candidate weights
    // sum to one), so this is the same interpolation, but float now resolves
    // the small differences u +- p/(rho c) that carry the pressure in a liquid.
    constexpr bool DELTA = sizeof(R) != sizeof(double);
    // Float faces and the learned weights (whose inputs are bfloat16) round
    // doubles to fewer bits: they keep the order of operations that their results
    // stand for
    constexpr bool KEPT = DELTA || WT == 1;
    auto nv = [&](int j, int f) -> R { return (R)nodev<NS, FS>(nd, j, f); };
    auto dv = [&](int j, int f) -> R {
        return DELTA ? (R)(nodev<NS, FS>(nd, j, f) - nodev<NS, FS>(nd, 2, f)) : (R)nodev<NS, FS>(nd, j, f);
    };
    auto back = [&](int f, R d) -> R { return DELTA ? (R)(nodev<NS, FS>(nd, 2, f) + (double)d) : d; };
    auto back_d = [&](int f, R d) -> double { return DELTA ? nodev<NS, FS>(nd, 2, f) + (double)d : (double)d; };

    // the two nodes of the face (i, i+1), read from LDS where they are used:
    // the compiler barrier forces fresh reads, so the node states do not
    // occupy registers across the whole face computation
    auto node_pair = [&](St<N, D>& a, St<N, D>& b) {
        asm volatile("" ::: "memory");
        load_node<N, D, NS, FS>(nd, 2, a);
        load_node<N, D, NS, FS>(nd, 3, b);
    };

    // first-order HLLC of the node pair and its quasi-conservative pair
    // (eq:G_pm); needed only by the first-order scheme and by the flux
    // limiter when it has to act, so it is formed on demand
    auto first_order = [&](const St<N, D>& L, const St<N, D>& Rn, double* Glo, double* Glo_p) {
        const St<N, D, R> Lr = convert<N, D, R>(L), Rr = convert<N, D, R>(Rn);
        double ss;
        if constexpr (KEPT)
            ss = hllc_kept<N, D, DIR, R, true>(Lr, Rr, Glo);
        else
            ss = hllc<N, D, DIR>(Lr, Rr, Glo);
#pragma unroll
        for (int k = 0; k < N - 1; ++k) {
#pragma clang fp contract(off)
            Glo_p[k] = KEPT ? Glo[IA + k] - ss * Rr.al[k] : fma(-ss, Rr.al[k], Glo[IA + k]);
            Glo[IA + k] = fma(-ss, Lr.al[k], Glo[IA + k]);
        }
    };
    const int flags = kload<ParDev>(kp).flags;
    if (LOW == 2 || (LOW && (flags & F_FIRST_ORDER))) {
        St<N, D> L, Rn;
        node_pair(L, Rn);
        if (flags & F_FOUR_EQ) {
            // the four-equation HRM solved directly: the same solver on
            // (alpha_k rho_k, rho u, E); the node records hold the HRM pressure
            // and sound speed, and the volume fractions are not evolved
            hllc<N, D, DIR>(L, Rn, G);
#pragma unroll
            for (int k = 0; k < N - 1; ++k) G[IA + k] = Gp[k] = 0.0;
            return;
        }
        double Glo[M], Glo_p[NA];
        first_order(L, Rn, Glo, Glo_p);
#pragma unroll
        for (int c = 0; c < M; ++c) G[c] = Glo[c];
#pragma unroll
        for (int k = 0; k < N - 1; ++k) Gp[k] = Glo_p[k];
        return;
    }

    // App. D: projection with the midpoint means of alpha_k rho_k, rho and c
    R arb[N];
#pragma unroll
    for (int k = 0; k < N; ++k) arb[k] = (R)0.5 * (nv(2, k) + nv(3, k));
    const R rb = (R)0.5 * ((R)nodev<NS, FS>(nd, 2, F::RHO) + (R)nodev<NS, FS>(nd, 3, F::RHO));
    const R cb = (R)0.5 * (nv(2, F::C) + nv(3, F::C));
    // 1/(rho c), 1/(rho c^2) = rho (1/(rho c))^2 and 1/(2c) = rho/(2 rho c) from one
    // reciprocal (the means of two admissible nodes are positive)
    R irc;
    if constexpr (sizeof(R) == sizeof(double))
        irc = rcp_newton(rb * cb);
    else
        irc = div_rn((R)1, rb * cb);
    const R irc2 = irc * irc * rb;
    const ParDev Pw = kload<ParDev>(kp);
    const double eps = Pw.eps_weno;
    // The characteristic fields are interpolated one at a time and each is
    // taken back to its primitive slot (V = R U) at once, so that only the
    // two acoustic fields stay live across the others.
    St<N, D, R> VL, VR;
    const R h2c = (R)0.5 * rb * irc, hrc = (R)0.5 * rb * cb;
    R v[6], aL0, aR0, aLM, aRM;
#pragma unroll
    for (int j = 0; j < 6; ++j) v[j] = dv(j, F::U + DIR) - dv(j, F::P) * irc;
    interp_pair<R, WT>(v, eps, Pw.mlp, aL0, aR0);
#pragma unroll
    for (int j = 0; j < 6; ++j) v[j] = dv(j, F::U + DIR) + dv(j, F::P) * irc;
    interp_pair<R, WT>(v, eps, Pw.mlp, aLM, aRM);
    const R dUL = aLM - aL0, dUR = aRM - aR0;
    VL.u[DIR] = back(F::U + DIR, (R)0.5 * (aL0 + aLM));
    VR.u[DIR] = back(F::U + DIR, (R)0.5 * (aR0 + aRM));
    VL.p = back(F::P, hrc * dUL);
    VR.p = back(F::P, hrc * dUR);
#pragma unroll
    for (int k = 0; k < N; ++k) {
        const R s = arb[k] * irc2;
#pragma unroll
        for (int j = 0; j < 6; ++j) v[j] = dv(j, k) - s * dv(j, F::P);
        R l, r;
        interp_pair<R, WT>(v, eps, Pw.mlp, l, r);
        VL.ar[k] = back(k, l + arb[k] * h2c * dUL);
        VR.ar[k] = back(k, r + arb[k] * h2c * dUR);
    }
#pragma unroll
    for (int d = 0; d < D; ++d) {
        if (d == DIR) continue;
#pragma unroll
        for (int j = 0; j < 6; ++j) v[j] = dv(j, F::U + d);
        R l, r;
        interp_pair<R, WT>(v, eps, Pw.mlp, l, r);
        VL.u[d] = back(F::U + d, l);
        VR.u[d] = back(F::U + d, r);
    }
#pragma unroll
    for (int k = 0; k < N - 1; ++k) {
#pragma unroll
        for (int j = 0; j < 6; ++j) v[j] = dv(j, IA + k);
        R l, r;
        interp_pair<R, WT>(v, eps, Pw.mlp, l, r);
        VL.al[k] = back_d(IA + k, l);
        VR.al[k] = back_d(IA + k, r);
    }

    // Sec. 4.3.2 interpolation limiter: left against node i, right against node i+1
    if (!(flags & F_NO_LIMITERS)) {
        const bool cl = interp_clean<N, D, DIR, R>(ke, kp, VL), cr = interp_clean<N, D, DIR, R>(ke, kp, VR);
        if (__builtin_expect(!(cl & cr), 0)) {
            St<N, D> L, Rn;
            node_pair(L, Rn);
            set_rc2<N, D>(ke, L);
            set_rc2<N, D>(ke, Rn);
            interp_limit<N, D, DIR, R>(ke, kp, VL, convert<N, D, R>(L), cnt);  // also completes the state
            interp_limit<N, D, DIR, R>(ke, kp, VR, convert<N, D, R>(Rn), cnt);
        }
    } else {
        const EosDev e = kload<EosDev>(ke);
        complete_from_prim<N, D, R, DIR>(e, VL);
        complete_from_prim<N, D, R, DIR>(e, VR);
    }

    // midpoint flux and velocity from HLLC on the interpolated states
    double Gt[M];
    R ut;
    if constexpr (KEPT)
        ut = hllc_kept<N, D, DIR, R>(VL, VR, Gt);
    else
        ut = hllc<N, D, DIR>(VL, VR, Gt);

    // shock sensor (Sec. 4.3.1) on mixture density and pressure, in double in
    // both variants: C_s = 1e12 turns float rounding of p at a contact into
    // a visible blending weight
    const ParDev P = kload<ParDev>(kp);
    R sig = 0;
    if (!(flags & F_NO_BLEND)) {
        double r[6], pr[6];
#pragma unroll
        for (int j = 0; j < 6; ++j) {
            r[j] = nodev<NS, FS>(nd, j, F::RHO);
            pr[j] = nodev<NS, FS>(nd, j, F::P);
        }
        const double z = KEPT ? sensor_product_kept(r, pr) : sensor_product(r, pr);
        const double arg = P.Cs * (P.qexp == 2.0 ? z * z : pow(z, P.qexp));
        // tanh is exactly 0 at 0 and rounds to 1 for arguments >= 22; below
        // 0.01 (smooth flow: nearly every face) its odd series to x^7 is
        // exact to double rounding (the next term is below 3e-18 x)
        double th;
        if (arg < 0.01) {
            const double a2 = arg * arg;
            th = arg * (1.0 + a2 * (-1.0 / 3.0 + a2 * (2.0 / 15.0 - a2 * (17.0 / 315.0))));
        } else {
            th = arg >= 22.0 ? 1.0 : tanh(arg);
        }
        sig = (R)th;
    }

    // HCS reconstruction (eq:reconstructed_G, eq:reconstructed_vel) and blending.
    // Volume-fraction slots and the face velocity u-hat are double in both
    // variants: G^+-_alpha = G_alpha - u-hat alpha_i cancels to (alpha-tilde -
    // alpha_i) u-hat only if both terms see the same velocity at full precision.
    double Gho[M], Gho_p[NA], uh;
    if constexpr (!KEPT) {
        // every slot's flux at node j is its conserved value times u_j (plus
        // pressure terms), so the node weights of the reconstruction are
        // multiplied into u_j once and each slot is six multiply-adds
        const double wt[6] = {-P.hcs_c, P.hcs_b, -P.hcs_a, -P.hcs_a, P.hcs_b, -P.hcs_c};
        double cu[6], pw = 0.0, epw = 0.0;
        uh = P.psi * ut;
#pragma unroll
        for (int j = 0; j < 6; ++j) {
            cu[j] = wt[j] * nodev<NS, FS>(nd, j, F::U + DIR);
            const double pj = nodev<NS, FS>(nd, j, F::P);
            uh += cu[j];
            pw = fma(wt[j], pj, pw);
            epw = fma(cu[j], pj, epw);
        }
        const double om = 1.0 - sig;  // 0 where the sensor is 1: nothing of h is left then
        uh = fma(sig, ut, om * uh);
#pragma unroll
        for (int c = 0; c < M; ++c) {
            double h = P.psi * Gt[c];
            if (c == N + DIR) h += pw;
            if (c == IE) h += epw;
#pragma unroll
            for (int j = 0; j < 6; ++j) h = fma(cu[j], nodev<NS, FS>(nd, j, c), h);
            Gho[c] = fma(sig, Gt[c], om * h);
        }
    } else {
        R un[6], pj[6];
        double und[6];
#pragma unroll
        for (int j = 0; j < 6; ++j) {
            und[j] = nodev<NS, FS>(nd, j, F::U + DIR);
            un[j] = (R)und[j];
            pj[j] = nv(j, F::P);
        }
        const double sigd = sig;
#pragma unroll
        for (int c = 0; c < M; ++c) {
            if (c >= IA) {
                auto pair = [&](int i, int j) {
#pragma clang fp contract(off)
                    return fma(nodev<NS, FS>(nd, i, c), und[i], nodev<NS, FS>(nd, j, c) * und[j]);
                };
                Gho[c] = hcs_blend(P, sigd, Gt[c], pair(2, 3), pair(1, 4), pair(0, 5));
            } else {
                auto pair = [&](int i, int j) -> R {
#pragma clang fp contract(off)
                    const R wi = nv(i, c), wj = nv(j, c);
                    if (c == N + DIR) return fma(wi, un[i], pj[i]) + fma(wj, un[j], pj[j]);
                    if (c >= N && c < N + D) return wi * un[i] + wj * un[j];
                    if (c == IE) return fma(wi + pj[i], un[i], (wj + pj[j]) * un[j]);
                    if (WT == 1 && DIR == 0 && c == N - 2 && i == 2) return fma(wj, un[j], wi * un[i]);
                    return fma(wi, un[i], wj * un[j]);
                };
                Gho[c] = hcs_blend<R>(P, sig, (R)Gt[c], pair(2, 3), pair(1, 4), pair(0, 5));
            }
        }
        uh = hcs_blend(P, sigd, (double)ut, und[2] + und[3], und[1] + und[4], und[0] + und[5]);
    }

    // high-order quasi-conservative pair: alpha slots minus u-hat alpha_i / alpha_{i+1}
#pragma unroll
    for (int k = 0; k < N - 1; ++k) {
        Gho_p[k] = fma(-uh, nodev<NS, FS>(nd, 3, IA + k), Gho[IA + k]);
        Gho[IA + k] = fma(-uh, nodev<NS, FS>(nd, 2, IA + k), Gho[IA + k]);
    }
    if (flags & F_NO_LIMITERS) {
#pragma unroll
        for (int c = 0; c < M; ++c) G[c] = Gho[c];
#pragma unroll
        for (int k = 0; k < N - 1; ++k) Gp[k] = Gho_p[k];
        return;
    }
    // Alg. 3 and Alg. 4 leave the high-order pair untouched when its half-cell
    // states already satisfy every bound (the usual case away from
    // interfaces and shocks); the first-order pair is formed only otherwise
    St<N, D> L, Rn;
    node_pair(L, Rn);
    if (flux_limit_clean<N, D, DIR>(ke, kp, L, Rn, lam, Gho, Gho_p)) {
#pragma unroll
        for (int c = 0; c < M; ++c) G[c] = Gho[c];
#pragma unroll
        for (int k = 0; k < N - 1; ++k) Gp[k] = Gho_p[k];
        return;
    }
    // In double, the full limiter reads the node pair afresh (the same
    // values): products of the check above are then not kept for it, and the
    // usual path carries no registers (spilled, at this pressure) into the
    // rare one.  256^3 FP64 step -4 %; the float variant, which spills less,
    // measured 1 % slower with it.
    St<N, D> Lf = L, Rf = Rn;
    if constexpr (sizeof(R) == sizeof(double)) node_pair(Lf, Rf);
    double Glo[M], Glo_p[NA];
    first_order(Lf, Rf, Glo, Glo_p);
    flux_limit<N, D, DIR, DELTA>(ke, kp, Lf, Rf, lam, Gho, Gho_p, Glo, Glo_p, G, Gp, cnt);
}

}  // namespace hrm
