// kbc_device.hpp -- per-node arithmetic of the D2Q9 KBC / LBGK step for gfx950.
//
// The collision works on deviations g_i = f_i - W_i rho0 (the stored form) and
// never forms full populations.  Everything it needs follows from six
// non-equilibrium moments of df = f - feq, which are cheap in deviation form
// because the second-order polynomial equilibrium (eq. Eq) has closed-form
// moments on D2Q9: rho, rho u, Pi^eq = rho cs2 I + rho u u (eq. Peq),
// Q^eq_xyy = rho u_x / 3, Q^eq_yxx = rho u_y / 3 (eq. Qeq) and
// A^eq = rho / 9 + rho |u|^2 / 3.  With T = P_xx + P_yy, N = P_xx - P_yy,
// Pi = P_xy (eq. natmoments1), the shear part ds and the higher-order part dh
// of Table kbc_moment_grouping are populations of a moment vector
// (T, N, Pi, Q_xyy, Q_yxx, A) through eq. (momentsD2Q9); for the central-moment
// models A and B the shear moments are carried to natural ones by the linear
// part of eq. (cm) (at fixed u the central deviations equal the natural ones).
// gamma follows eq. (result21) with the entropic scalar product weighted by
// 1/feq; the common factor 1/rho cancels in the ratio and in the guard.
//
// All floating-point contractions are written out with fma() and the library
// is compiled with -ffp-contract=off, so every launch shape that runs this
// code produces bitwise identical results.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace kbc {

enum Coll { LBGK = 0, KBCC = 1 };
enum Var { VA = 0, VB = 1, VC = 2, VD = 3 };
enum GMode { GEST = 0, GFIX = 1, GEXACT = 2 };
enum FormId { F16 = 0, F32 = 1, F64 = 2 };

// D2Q9 velocities, order (0,0) (1,0) (0,1) (-1,0) (0,-1) (1,1) (-1,1) (-1,-1) (1,-1)
constexpr int kCx[9] = {0, 1, 0, -1, 0, 1, -1, -1, 1};
constexpr int kCy[9] = {0, 0, 1, 0, -1, 1, 1, -1, -1};
// lattice weights 4/9, 1/9, 1/36
__host__ __device__ constexpr double weight(int i) { return i == 0 ? 4.0 / 9.0 : (i < 5 ? 1.0 / 9.0 : 1.0 / 36.0); }
// binary16 storage scale exponents: ~1/W_i rounded to a power of two
__host__ __device__ constexpr int f16_shift(int i) { return i == 0 ? 1 : (i < 5 ? 3 : 5); }

// ---------------------------------------------------------------- storage forms
template <int FORM> struct Form;

template <> struct Form<F16> {
    using S = _Float16;
    using R = float;
    static constexpr int bytes = 2;
    // v 2^-s as one mixed-precision FMA (binary16 operand, binary32 result;
    // exact: the scale is a power of two).  The +0 addend keeps the FMA from
    // being rewritten as a conversion and a multiply; it maps a stored -0 to
    // +0, which no later sum can tell apart.
    __device__ static __forceinline__ R dec(S v, int i) {
        return __builtin_fmaf(static_cast<float>(v), 1.0f / static_cast<float>(1 << f16_shift(i)), 0.0f);
    }
    __device__ static __forceinline__ double dec64(S v, int i) {
        return static_cast<double>(static_cast<float>(v)) / static_cast<double>(1 << f16_shift(i));
    }
    // one rounding, double -> binary16 (not through binary32, which would
    // round twice and can land one unit away)
    __device__ static __forceinline__ S enc64(double v, int i) {
        return static_cast<_Float16>(v * static_cast<double>(1 << f16_shift(i)));
    }
};

template <> struct Form<F32> {
    using S = float;
    using R = float;
    static constexpr int bytes = 4;
    __device__ static __forceinline__ R dec(S v, int) { return v; }
    __device__ static __forceinline__ double dec64(S v, int) { return static_cast<double>(v); }
    __device__ static __forceinline__ S enc64(double v, int) { return static_cast<float>(v); }
};

template <> struct Form<F64> {
    using S = double;
    using R = double;
    static constexpr int bytes = 8;
    __device__ static __forceinline__ R dec(S v, int) { return v; }
    __device__ static __forceinline__ double dec64(S v, int) { return v; }
    __device__ static __forceinline__ S enc64(double v, int) { return v; }
};

// ------------------------------------------------------------------- arithmetic
__device__ __forceinline__ float fmaR(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fmaR(double a, double b, double c) { return __builtin_fma(a, b, c); }
// reciprocal: v_rcp_f32 (1 ulp) in FP32; in FP64 v_rcp_f64 (good to 2^-24)
// refined by one third-order step r <- r + r (e + e^2), e = 1 - a r, which
// leaves e^3 = 2^-72: three FMAs where two Newton steps take four, and one
// fewer in a row (without the scaling and final correction of the compiler's
// own division: within about an ulp for the positive normal denominators used
// here).  Of 2^22 arguments in [1/64, 8) both leave the same 1026 not correctly
// rounded, none by more than 2^-53.
__device__ __forceinline__ float rcpR(float a) { return __builtin_amdgcn_rcpf(a); }
__device__ __forceinline__ double rcpR(double a) {
    const double r = __builtin_amdgcn_rcp(a), e = __builtin_fma(-a, r, 1.0);
    return __builtin_fma(r, __builtin_fma(e, e, e), r);
}
__device__ __forceinline__ float divR(float a, float b) { return a * __builtin_amdgcn_rcpf(b); }
__device__ __forceinline__ double divR(double a, double b) { return a * rcpR(b); }

template <typename R> struct Coef {
    R beta;            // relaxation parameter
    R inv_beta;        // 1 / beta
    R two_m_inv_beta;  // 2 - 1 / beta
    R rho0;            // reference density of the deviation storage
    R guard;           // gamma = 2 where <dh|dh> <= guard <ds|ds>
    R gamma_fixed;     // stabiliser for GFIX
};

// ln(1 + x) for x > -1.  FP32: Goldberg's form (D. Goldberg, "What every
// computer scientist should know about floating-point arithmetic", 1991,
// Theorem 4): with u = fl(1 + x), ln(u) x / (u - 1) is accurate to a few
// units in the last place, because the rounding error of 1 + x cancels
// between ln(u) and u - 1; ln(u) comes from the hardware base-2 logarithm
// (about 10 instructions instead of the library's long compensated form).
// FP64 keeps the library log1p.
__device__ __forceinline__ float log1pR(float x) {
    const float u = 1.0f + x;
    const float d = u - 1.0f;
    return d == 0.0f ? x : (__builtin_amdgcn_logf(u) * 0.693147180559945309f) * (x * __builtin_amdgcn_rcpf(d));
}
__device__ __forceinline__ double log1pR(double x) { return log1p(x); }

// Forward quantities of one KBC collision at a node, shared by the step
// (collide) and its adjoint (collide_vjp) so that both take the same
// decisions on the same values.
//
// ds, dh and w are kept in scaled units: the rest population's parts at half
// their value and the diagonals' at twice (node_scale), their weights at four
// times and a quarter (1 / node_scale^2), so that ds_i dh_i w_i is unchanged.  In
// these units the populations of ds and dh are plain sums of the moments (no
// multiplications by 1/4, 1/2, 2, 4), the nine denominators of the weights
// share their leading terms, and the rest population's denominator is one of
// those terms.
template <typename R> struct KbcNode {
    R dr, rho, ir, jx, jy;              // rho - rho0, rho, 1 / rho, rho u
    R ux, uy, uxx, u2;
    R dT, dN, dP;                       // non-equilibrium T, N, Pi
    R tpn, tmn, ox, oy;                 // of the shear part: (T_s +- N) / 4, Q_xyy,s / 2, Q_yxx,s / 2
    R ds[9], dh[9];                     // shear and higher-order parts of f - feq (scaled)
    R w[9];                             // rho / feq_i (entropic weights, scaled)
    R ratio, b;                         // <ds|dh> / <dh|dh> and <dh|dh>
    R gam;                              // stabiliser used (estimate, 2 when guarded, or fixed)
    bool active;                        // gamma follows eq. (result21) (not guarded, not fixed)
};
template <typename R> constexpr R node_scale(int i) { return i == 0 ? R(0.5) : (i < 5 ? R(1) : R(2)); }

// <ds|ds> of the guard is compared only where <dh|dh> is small: with
// |u|^2 < 1/6 every 1 + e_i is at least 1/4 (3 c.u + 4.5 (c.u)^2 >= -1/2), so
// 1 / (W_i (1 + e_i)) <= 4 / W_i, and with the bounds of |ds_i| in the moments
// (|Q| <= 0.82 |Pi| + 0.21 (|T| + |N|), |A| <= 0.34 |Pi| + 0.084 (|T| + |N|))
// <ds|ds> <= 1110 Pi^2 + 128 T^2 + 98 N^2; the constant leaves room for rounding.
template <typename R> constexpr R guard_bound() { return R(1300); }

// Written for instruction count: the kernels that call it issue one vector
// instruction per operation here and are bound by that issue rate, so every
// product-plus-sum is an explicit FMA (contraction is off) and scale factors
// are folded into the moments before they are spread back to populations.
// FP32 KBC-B takes 151 vector instructions per collision (181 with unscaled
// populations spread one by one and <ds|ds> always formed).  The fused step of
// an FP16 lattice, bound by instruction issue, went from 35.1 to 31.8 us per
// pair of steps at 1921 x 1083 with it, of FP64 2-3 %; FP32 at 8192^2 from 975
// to 918, where it moves 5.3 TB/s and is bound by memory as much.
// The natural-moment variants (C, D) sum in the order that has been checked
// over 2000-step gradients: there too every scale is a power of two.
//
// The populations come as sums and differences of opposite ones (PopSums).
// They may be given in units of their own: U times the axis populations and
// U Q times the diagonal ones (powers of two; U = Q = 1 for plain values).  All
// of n is then in units of U (every moment is homogeneous in the deviations
// and rho0, and velocities, weights, gamma and the guard have no unit), with
// the factors 1 / Q in multiplications that are there anyway.
template <typename R> struct PopSums {
    R s13, s24, s57, s68;               // g1 + g3, ...
    R d13, d24, d57, d68;               // g1 - g3, ...
};
template <typename R>
__device__ __forceinline__ PopSums<R> pop_sums(const R (&g)[9]) {
    return {g[1] + g[3], g[2] + g[4], g[5] + g[7], g[6] + g[8], g[1] - g[3], g[2] - g[4], g[5] - g[7], g[6] - g[8]};
}
template <typename R, int VAR, int GM, int U, int Q, typename Rest>
__device__ __forceinline__ void kbc_forward_sums(const PopSums<R>& p, Rest add_rest, const Coef<R>& K,
                                                 KbcNode<R>& n) {
    constexpr bool kCentral = (VAR == VA || VAR == VB);   // s in the co-moving frame, eq. (cm)
    constexpr bool kTrace = (VAR == VA || VAR == VC);     // T belongs to s
    constexpr R q = R(1) / R(Q);
    auto plus = [](R a, R b) { return Q == 1 ? a + b : fmaR(q, b, a); };   // a + q b
    // conserved moments, eq. (moments) restricted to the deviations
    const R s13 = p.s13, s24 = p.s24, s57 = p.s57, s68 = p.s68;
    const R d13 = p.d13, d24 = p.d24;
    const R sd = s57 + s68, sa = s13 + s24;
    const R dr = plus(sa, add_rest(sd));           // rho - rho0
    const R mq = p.d57 - p.d68, pq = p.d57 + p.d68;
    const R jx = plus(d13, mq);                    // rho u_x
    const R jy = plus(d24, pq);                    // rho u_y
    const R rho = U == 1 ? K.rho0 + dr : fmaR(R(U), K.rho0, dr);
    const R ir = rcpR(rho);
    const R ux = jx * ir, uy = jy * ir;
    const R uxx = ux * ux, uyy = uy * uy;
    const R u2 = kCentral ? fmaR(uy, uy, uxx) : uxx + uyy;
    n.dr = dr; n.rho = rho; n.ir = ir; n.jx = jx; n.jy = jy;
    n.ux = ux; n.uy = uy; n.uxx = uxx; n.u2 = u2;

    // non-equilibrium moments of df = f - feq (feq of second order, c_s^2 = 1/3)
    const R juy = jy * uy;
    const R jsum = fmaR(jx, ux, juy);          // rho |u|^2
    const R jdif = fmaR(jx, ux, -juy);         // rho (u_x^2 - u_y^2)
    const R dT = fmaR(R(2) * q, sd, sa) - fmaR(R(2.0 / 3.0), dr, jsum);
    const R dN = (s13 - s24) - jdif;
    const R dP = fmaR(-jx, uy, Q == 1 ? s57 - s68 : q * (s57 - s68));
    const R dQx = fmaR(R(-Q / 3.0), jx, mq);       // Q times dQ_xyy, dQ_yxx and dA
    const R dQy = fmaR(R(-Q / 3.0), jy, pq);
    const R dA = fmaR(R(-Q / 3.0), jsum, fmaR(R(-Q / 9.0), dr, sd));
    constexpr R hq = R(0.5) * q;
    n.dT = dT; n.dN = dN; n.dP = dP;

    // Shear part s, Table kbc_moment_grouping, from (T_s +- N) / 4, Q_xyy,s / 2
    // (ox), Q_yxx,s / 2 (oy) and A_s / 2 (a2).  Central variants take the
    // linear part of eq. (cm) at the node's velocity, in which
    // A_s = u_x Q_xyy,s + u_y Q_yxx,s.
    const R n4 = R(0.25) * dN;
    const R tq = R(0.25) * dT;
    const R tpn = kTrace ? tq + n4 : n4, tmn = kTrace ? tq - n4 : -n4;
    const R p2 = R(0.5) * dP;
    n.tpn = tpn;
    n.tmn = tmn;
    R (&ds)[9] = n.ds;
    R ox = R(0), oy = R(0), a2 = R(0);
    if constexpr (kCentral) {
        ox = fmaR(uy, dP, ux * tmn);
        oy = fmaR(ux, dP, uy * tpn);
        a2 = fmaR(ux, ox, uy * oy);
        n.ox = ox;
        n.oy = oy;
        const R e1 = tpn - a2, e2 = tmn - a2;
        ds[0] = kTrace ? fmaR(R(-0.5), dT, a2) : a2;
        ds[1] = e1 - ox;
        ds[3] = e1 + ox;
        ds[2] = e2 - oy;
        ds[4] = e2 + oy;
        const R ap = a2 + p2, am = a2 - p2, xp = ox + oy, xm = ox - oy;
        ds[5] = ap + xp;
        ds[7] = ap - xp;
        ds[6] = am - xm;
        ds[8] = am + xm;
    } else {
        ds[0] = kTrace ? R(-0.5) * dT : R(0);
        ds[1] = tpn;
        ds[3] = tpn;
        ds[2] = tmn;
        ds[4] = tmn;
        ds[5] = p2;
        ds[7] = p2;
        ds[6] = -p2;
        ds[8] = -p2;
    }
    // higher-order part h = df - s: moments (T - T_s, 0, 0, dQ - Q_s, dA - A_s)
    R (&dh)[9] = n.dh;
    {
        const R xh = kCentral ? fmaR(hq, dQx, -ox) : hq * dQx;
        const R yh = kCentral ? fmaR(hq, dQy, -oy) : hq * dQy;
        const R ah = kCentral ? fmaR(hq, dA, -a2) : hq * dA;
        dh[0] = kTrace ? ah : fmaR(R(-0.5), dT, ah);
        if constexpr (kCentral) {
            const R eh = kTrace ? -ah : tq - ah;
            dh[1] = eh - xh;
            dh[3] = eh + xh;
            dh[2] = eh - yh;
            dh[4] = eh + yh;
        } else {
            dh[1] = kTrace ? -(xh + ah) : tq - (xh + ah);
            dh[3] = kTrace ? xh - ah : tq + (xh - ah);
            dh[2] = kTrace ? -(yh + ah) : tq - (yh + ah);
            dh[4] = kTrace ? yh - ah : tq + (yh - ah);
        }
        const R hp = xh + yh, hm = xh - yh;
        dh[5] = ah + hp;
        dh[7] = ah - hp;
        dh[6] = ah - hm;
        dh[8] = ah + hm;
    }

    if constexpr (GM == GFIX) {
        n.gam = K.gamma_fixed;
        n.active = false;
        n.ratio = R(0);
        n.b = R(1);
    } else {
        // entropic scalar products, weights 1 / (W_i (1 + e_i)) = rho / feq_i;
        // d_i = W_i (1 + e_i) = W_i (1 - 1.5 |u|^2 + 4.5 (v.u)^2) + 3 W_i (v.u),
        // a quarter of it for the rest population and four times for the diagonals
        const R upv = ux + uy, umv = ux - uy;
        const R a1 = fmaR(R(-1.0 / 6.0), u2, R(1.0 / 9.0));
        const R b1 = fmaR(R(1.0 / 3.0), u2, R(1.0 / 9.0));
        const R uxy = ux * uy;
        const R dx = fmaR(R(0.5), uxx, a1), dy = kCentral ? fmaR(R(-0.5), uxx, b1) : fmaR(R(0.5), uyy, a1);
        const R dp = kCentral ? fmaR(ux, uy, b1) : b1 + uxy, dm = kCentral ? fmaR(-ux, uy, b1) : b1 - uxy;
        R d[9];
        d[0] = a1;
        d[1] = fmaR(R(1.0 / 3.0), ux, dx);
        d[3] = fmaR(R(-1.0 / 3.0), ux, dx);
        d[2] = fmaR(R(1.0 / 3.0), uy, dy);
        d[4] = fmaR(R(-1.0 / 3.0), uy, dy);
        d[5] = fmaR(R(1.0 / 3.0), upv, dp);
        d[7] = fmaR(R(-1.0 / 3.0), upv, dp);
        d[8] = fmaR(R(1.0 / 3.0), umv, dm);
        d[6] = fmaR(R(-1.0 / 3.0), umv, dm);
        R a = R(0), b = R(0);
        R wh[9];
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            n.w[i] = rcpR(d[i]);
            wh[i] = dh[i] * n.w[i];
            b = i ? fmaR(dh[i], wh[i], b) : dh[i] * wh[i];
            if (VAR != VD || i) a = (i == (VAR == VD ? 1 : 0)) ? ds[i] * wh[i] : fmaR(ds[i], wh[i], a);
        }
        n.ratio = divR(a, b);
        n.b = b;
        const R gs = fmaR(-K.two_m_inv_beta, n.ratio, K.inv_beta);
        // the guard, eq. (result21) only where <dh|dh> > guard <ds|ds>
        if constexpr (kCentral) {
            // <ds|ds> (18 instructions) is formed by the waves that hold a
            // node where its bound does not decide (or a NaN)
            R m = fmaR(dP, dP, dN * dN);
            if constexpr (kTrace) m = fmaR(dT, dT, m);
            n.active = true;
            if (!(b > (guard_bound<R>() * K.guard) * m && u2 < R(1.0 / 6.0))) {
                R c = R(0);
#pragma unroll
                for (int i = 0; i < 9; ++i) c = fmaR(ds[i] * n.w[i], ds[i], c);
                n.active = !(b <= K.guard * c);
            }
        } else {
            // populations of ds that differ in sign only are summed by their weights
            const R wd = (n.w[5] + n.w[7]) + (n.w[6] + n.w[8]);
            const R wx = n.w[1] + n.w[3], wy = n.w[2] + n.w[4];
            R c;
            if constexpr (kTrace) {
                c = fmaR(p2 * p2, wd, fmaR(tpn * tpn, wx, (tmn * tmn) * wy));
                c = fmaR(ds[0] * n.w[0], ds[0], c);
            } else {
                c = fmaR(p2 * p2, wd, (n4 * n4) * (wx + wy));
            }
            n.active = !(b <= K.guard * c);
        }
        n.gam = n.active ? gs : R(2);
    }
}

// The node's quantities from its deviations g.
template <typename R, int VAR, int GM>
__device__ __forceinline__ void kbc_forward(const R (&g)[9], const Coef<R>& K, KbcNode<R>& n) {
    kbc_forward_sums<R, VAR, GM, 1, 1>(pop_sums(g), [&](R sd) { return g[0] + sd; }, K, n);
}

// Root of the entropy-maximum condition eq. (result1) in gamma,
//   F(gamma) = sum_i dh_i ln(1 + x_i) = 0,
//   x_i = ((1 - beta gamma) dh_i - (2 beta - 1) ds_i) / feq_i,
// by iteration from gamma* (its first-order root, eq. (result21)).
// F decreases strictly in gamma while every 1 + x_i > 0, so the root is
// unique; the iteration stops (keeping the current gamma) if an argument of
// the logarithm leaves (0, inf) or F' is not negative, after a step below
// the tolerance of the arithmetic type, after a step that is not at most half
// the previous one (Newton's steps shrink quadratically until rounding noise
// in F takes over, which at a near-equilibrium node lies above the FP32
// tolerance), or after a fixed number of steps.
// 1 / feq_i = w_i / rho with w_i = 1 / (W_i (1 + e_i)); ln(1 + x) is taken
// as log1pR(x), accurate to rounding for the small x of a near-equilibrium
// node.
//
// While every |x_i| of a node is below 1/32 (FP32) or 1/64 (FP64), i.e. near
// equilibrium, ln(1 + x) is its Taylor polynomial, of degree 6 or 10, by
// Horner's rule: six or ten FMAs against the general form's logarithm,
// reciprocal and guard (FP32) or the library log1p (FP64).  The truncation is
// below 1.4e-10 and 8e-20 relative, the evaluation within 1.2e-7 and 1.5 ulp.
// Above that and up to 1/2 the FP64 logarithm is log1p_mid; the library's (about
// 100 instructions, nine times an iteration) is left to nodes beyond.  A few
// such nodes set the time of their waves: 300 x 217 FP64 KBC-B 62 -> 8 us per
// step, 1024^2 269 -> 77 (with the third-order steps below).  The
// choice is the node's own (all nine of its arguments small), so a node's
// result does not depend on which nodes share its wave; a wave skips the
// general form when none of its nodes needs it.  The quantities that do not change
// with gamma (dh_i / feq_i, (2 beta - 1) ds_i / feq_i) are formed once, before
// the iteration.
//
// In that regime a step is not Newton's but third order (Schroeder's method:
// the inverse series of F).  With q_i = (dh_i / feq_i) / (1 + x_i) and
// A_k = sum_i dh_i q_i^k, all of which come with the evaluation of F,
//   F(gamma + eta / beta) = F - A_1 eta - A_2 eta^2 / 2 - A_3 eta^3 / 3 - ...,
// so with e = F / A_1, u = A_2 e / (2 A_1), v = A_3 e^2 / (3 A_1) the root is at
//   eta = e (1 - u + 2 u^2 - v + O((e q)^3)).
// e q is of the order of x^2, so one evaluation (about 160 instructions) mostly
// does what three of Newton's (125 each) did; the iteration also stops when
// the third-order term itself is below the tolerance (what remains is smaller
// by another factor e q).  FP32 KBC-B, 1024^2, 10 steps: 140 us, 265 with
// Newton's.
__device__ __forceinline__ float log1p_small(float x) {
    float p = fmaR(x, -1.0f / 6.0f, 0.2f);
    p = fmaR(x, p, -0.25f);
    p = fmaR(x, p, 1.0f / 3.0f);
    p = fmaR(x, p, -0.5f);
    p = fmaR(x, p, 1.0f);
    return x * p;
}
// FP64: below 1/64 the Taylor polynomial of degree 10 (truncation below
// 8e-20 relative, evaluation within 1.5 ulp) replaces the library log1p
__device__ __forceinline__ double log1p_small(double x) {
    double p = fmaR(x, -1.0 / 10.0, 1.0 / 9.0);
    p = fmaR(x, p, -1.0 / 8.0);
    p = fmaR(x, p, 1.0 / 7.0);
    p = fmaR(x, p, -1.0 / 6.0);
    p = fmaR(x, p, 1.0 / 5.0);
    p = fmaR(x, p, -1.0 / 4.0);
    p = fmaR(x, p, 1.0 / 3.0);
    p = fmaR(x, p, -1.0 / 2.0);
    p = fmaR(x, p, 1.0);
    return x * p;
}
// atanh(s) = s P(s^2), P(z) = 1 + z T(z), for s^2 = z <= 1/9, i.e. logarithms
// 2 atanh(s) of arguments in [1/2, 2]: P the polynomial of degree 10 with the
// smallest largest relative error (coefficients by Remez's exchange algorithm;
// 2.5e-18 with the coefficients rounded as below).
__device__ __forceinline__ double atanh_tail(double z) {
    double p = 0.08504923007075064;
    p = fmaR(z, p, 0.04172462195061191);
    p = fmaR(z, p, 0.06052477641340325);
    p = fmaR(z, p, 0.06650560071689546);
    p = fmaR(z, p, 0.07693274239195039);
    p = fmaR(z, p, 0.09090872237804135);
    p = fmaR(z, p, 0.11111111976861492);
    p = fmaR(z, p, 0.14285714274058622);
    p = fmaR(z, p, 0.20000000000077559);
    return fmaR(z, p, 0.33333333333333154);
}
__device__ __forceinline__ double atanh_poly(double z) { return fmaR(z, atanh_tail(z), 1.0); }
// ln(1 + x) = 2 atanh(x / (2 + x)) for x in [-1/2, 1/2], given r = 1 / (2 + x) to
// a few units in the last place: within 0.56 ulp (0.83 for the host's library
// log1p).  The quotient is carried as s + sl, with tl the rounding error of
// t = 2 + x and sl the remainder x - s (t + tl) over t; the leading part 2 s is
// added last.  (With the quotient as the one product x r the error reaches 3.3
// ulp, and the 99th percentile of the error in gamma grows by 11 %.)  What that takes is
// mostly paid for by the one reciprocal that 1 / (1 + x) and 1 / (2 + x) share:
// 1024^2 FP64 KBC-B 75 -> 78 us per step.
__device__ __forceinline__ double log1p_mid(double x, double r) {
    const double t = 2.0 + x, tl = x - (t - 2.0), s = x * r;
    const double sl = fmaR(-s, tl, fmaR(-s, t, x)) * r;
    const double z = s * s;
    return fmaR(2.0, fmaR(s * z, atanh_tail(z), fmaR(z, sl, sl)), 2.0 * s);
}
__device__ __forceinline__ float log1p_mid(float x, float) { return log1pR(x); }
template <typename R> constexpr R log1p_mid_limit() { return sizeof(R) == 8 ? R(0.5) : R(0); }
template <typename R> constexpr R log1p_small_limit() { return sizeof(R) == 8 ? R(1.0 / 64.0) : R(1.0 / 32.0); }

// The iteration for the root.  It runs on t = beta gamma, which is what the
// collision multiplies dh by (returned in t): with gamma as the iterate the
// rounding of beta gamma comes on top, and near equilibrium, where an evaluation
// or two end the iteration, it raises the rms error of the populations (FP64
// KBC-D) to 1.10 .. 1.14 times that with the root correctly rounded, 1.01 with t.
// Returns gamma = t / beta.
template <typename R>
__device__ __forceinline__ R exact_gamma(const KbcNode<R>& n, const Coef<R>& K, R& t) {
    constexpr int kMaxIt = sizeof(R) == 8 ? 100 : 20;
    const R tol = sizeof(R) == 8 ? R(1e-15) : R(5e-7);
    const R tbm1 = R(2) * K.beta - R(1);
    t = K.beta * n.gam;
    R dh[9], hw[9], sw[9];   // dh_i, dh_i / feq_i, (2 beta - 1) ds_i / feq_i
    const R irs[3] = {R(0.5) * n.ir, n.ir, R(2) * n.ir};
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        const R wr = n.w[i] * irs[i == 0 ? 0 : (i < 5 ? 1 : 2)];
        hw[i] = n.dh[i] * wr;
        sw[i] = (tbm1 * n.ds[i]) * wr;
        dh[i] = (i == 0 || i > 4) ? n.dh[i] * (R(1) / node_scale<R>(i)) : n.dh[i];
    }
    R prev = R(1e30);   // size of the previous step
    for (int it = 0; it < kMaxIt; ++it) {
        const R om = R(1) - t;
        R x[9];
        R amax = R(0);
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            x[i] = fmaR(om, hw[i], -sw[i]);
            amax = fmax(amax, fabs(x[i]));
        }
        R step, rest;   // step in t; bound of what the step leaves, relative to it
        if (amax < log1p_small_limit<R>()) {
            R F = R(0), A1 = R(0), A2 = R(0), A3 = R(0);
#pragma unroll
            for (int i = 0; i < 9; ++i) {
                F = fmaR(dh[i], log1p_small(x[i]), F);
                const R q = hw[i] * rcpR(R(1) + x[i]);
                const R m = dh[i] * q, mq = m * q;
                A1 += m;
                A2 += mq;
                A3 = fmaR(mq, q, A3);
            }
            if (!(A1 > R(0))) break;
            const R ia = rcpR(A1);
            const R e1 = F * ia;
            const R u = R(0.5) * A2 * ia * e1, v = R(1.0 / 3.0) * A3 * ia * e1 * e1;
            const R uu = R(2) * u * u;
            const bool series = uu + v < R(1.0 / 64.0);
            step = series ? e1 * ((R(1) - u) + (uu - v)) : e1;
            rest = series ? uu + v : R(1);
        } else {
            bool ok = true;
            R F = R(0), D = R(0);
            if (amax <= log1p_mid_limit<R>()) {
                // one reciprocal for 1 / (1 + x) and 1 / (2 + x)
#pragma unroll
                for (int i = 0; i < 9; ++i) {
                    const R a = R(1) + x[i], b = R(2) + x[i], r = rcpR(a * b);
                    F = fmaR(dh[i], log1p_mid(x[i], a * r), F);
                    D = fmaR(-dh[i] * hw[i], b * r, D);
                }
            } else {
#pragma unroll
                for (int i = 0; i < 9; ++i) {
                    ok = ok && (x[i] > R(-1));
                    F = fmaR(dh[i], log1pR(x[i]), F);
                    D = fmaR(-dh[i] * hw[i], rcpR(R(1) + x[i]), D);
                }
            }
            if (!ok || !(D < R(0))) break;
            step = -divR(F, D);
            rest = R(1);
        }
        t += step;
        const R as = fabs(step);
        if (as * rest <= tol * fabs(t) || as > R(0.5) * prev) break;
        prev = as;
    }
    const R q = t * K.inv_beta;
    return fmaR(fmaR(-q, K.beta, t), K.inv_beta, q);
}

// ds, dh and w of a node in their own units.
template <typename R>
__device__ __forceinline__ void unscaled(const KbcNode<R>& n, R (&ds)[9], R (&dh)[9], R (&w)[9]) {
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        constexpr R one = R(1);
        const R k = one / node_scale<R>(i), k2 = node_scale<R>(i) * node_scale<R>(i);
        ds[i] = (i == 0 || i > 4) ? n.ds[i] * k : n.ds[i];
        dh[i] = (i == 0 || i > 4) ? n.dh[i] * k : n.dh[i];
        w[i] = (i == 0 || i > 4) ? n.w[i] * k2 : n.w[i];
    }
}

// One collision on a node's values (in place): U and Q are the units of the
// axis and diagonal ones (see PopSums) and Z that of the rest population, 1 / Z
// of the axis unit.  Returns the gamma used.
template <typename R, int COLL, int VAR, int GM, int U, int Q, int Z>
__device__ __forceinline__ R collide_units(R (&g)[9], const Coef<R>& K) {
    constexpr R rz = R(1) / R(Z);
    auto add_rest = [&](R sd) { return Q * Z == 1 ? g[0] + sd : fmaR(R(Q * Z), g[0], sd); };
    const PopSums<R> p = pop_sums(g);
    if constexpr (COLL == LBGK) {
        auto plus = [](R a, R b) { return Q == 1 ? a + b : fmaR(R(1) / R(Q), b, a); };
        const R dr = plus(p.s13 + p.s24, add_rest(p.s57 + p.s68));
        const R jx = plus(p.d13, p.d57 - p.d68), jy = plus(p.d24, p.d57 + p.d68);
        const R rho = U == 1 ? K.rho0 + dr : fmaR(R(U), K.rho0, dr);
        const R ir = rcpR(rho);
        const R ux = jx * ir, uy = jy * ir;
        const R uxx = ux * ux, uyy = uy * uy, u2 = uxx + uyy;
        const R upv = ux + uy, umv = ux - uy;
        // f' = f - 2 beta (f - feq), eq. (LBGKmirr) in eq. (Egeneral):
        // g' = (1 - 2 beta) g + 2 beta W_i [(rho - rho0) + rho e_i],
        // e_i = 3 (v.u) + 4.5 (v.u)^2 - 1.5 |u|^2
        const R c0 = R(-1.5) * u2;
        const R bx = fmaR(R(4.5), uxx, c0), by = fmaR(R(4.5), uyy, c0);
        const R uxy9 = R(9) * (ux * uy);
        const R b5 = fmaR(R(3), u2, uxy9), b6 = fmaR(R(3), u2, -uxy9);   // 4.5 (u_x +- u_y)^2 - 1.5 |u|^2
        R e[9];
        e[0] = c0;
        e[1] = fmaR(R(3), ux, bx);
        e[3] = fmaR(R(-3), ux, bx);
        e[2] = fmaR(R(3), uy, by);
        e[4] = fmaR(R(-3), uy, by);
        e[5] = fmaR(R(3), upv, b5);
        e[7] = fmaR(R(-3), upv, b5);
        e[8] = fmaR(R(3), umv, b6);
        e[6] = fmaR(R(-3), umv, b6);
        const R tb = R(2) * K.beta, omt = R(1) - tb;
        const R tw[3] = {tb * (R(weight(0)) * rz), tb * R(weight(1)), tb * (R(weight(5)) * R(Q))};
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            const R twi = tw[i == 0 ? 0 : (i < 5 ? 1 : 2)];
            g[i] = fmaR(omt, g[i], twi * fmaR(rho, e[i], dr));
        }
        return R(2);
    } else {
        KbcNode<R> n;
        kbc_forward_sums<R, VAR, (GM == GEXACT ? GEST : GM), U, Q>(p, add_rest, K, n);
        R gam = n.gam;
        R bgam = K.beta * gam;
        if constexpr (GM == GEXACT) {
            if (n.active) gam = exact_gamma<R>(n, K, bgam);
        }
        // f' = f - beta (2 ds + gamma dh), eqs. (Egeneral), (ksh-mirror)
        const R tb[3] = {(R(4) * rz) * K.beta, R(2) * K.beta, R(Q) * K.beta};
        R bg[3] = {((R(2) * rz) * K.beta) * gam, bgam, ((R(0.5) * R(Q)) * K.beta) * gam};
        if constexpr (GM == GEXACT) {
            bg[0] = (R(2) * rz) * bgam;
            bg[2] = (R(0.5) * R(Q)) * bgam;
        }
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            const int k = i == 0 ? 0 : (i < 5 ? 1 : 2);
            // D has no shear part in the rest population
            const R t = (VAR == VD && i == 0) ? g[0] : fmaR(-tb[k], n.ds[i], g[i]);
            g[i] = fmaR(-bg[k], n.dh[i], t);
        }
        return gam;
    }
}

// One collision on the deviations g (in place).  Returns the gamma used.
template <typename R, int COLL, int VAR, int GM>
__device__ __forceinline__ R collide(R (&g)[9], const Coef<R>& K) {
    return collide_units<R, COLL, VAR, GM, 1, 1, 1>(g, K);
}

// One collision on a node's values in the storage form (in place).
//
// FP16 works in the units the values are stored in (2^s_i g_i), so that a value
// is converted to binary32 and back and never scaled.  The conversions are kept
// apart from the arithmetic: folded into it as mixed-precision FMAs they are
// fewer instructions but slower ones (cycles per wave instruction among FP32
// FMAs, six waves per SIMD: v_cvt_f32_f16 and v_cvt_f16_f32 2.3, v_fma_f32 2.5,
// v_fma_mix_f32 4.5, v_fma_mixlo_f16 10.5, as much as a reciprocal).  KBC-B with
// mixed FMAs / conversions, us per launch: two steps at 1921 x 1083 34.0 / 31.2,
// four at 4096^2 409 / 382 (tiles of 32 rows).
template <int FORM, int COLL, int VAR, int GM>
__device__ __forceinline__ void collide_stored(typename Form<FORM>::S (&v)[9], const Coef<typename Form<FORM>::R>& K) {
    if constexpr (FORM == F16) {
        constexpr int sa = f16_shift(1);
        float g[9];
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            g[i] = static_cast<float>(v[i]);
            asm("" : "+v"(g[i]));
        }
        collide_units<float, COLL, VAR, GM, 1 << sa, 1 << (f16_shift(5) - sa), 1 << (sa - f16_shift(0))>(g, K);
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            asm("" : "+v"(g[i]));
            v[i] = static_cast<_Float16>(g[i]);
        }
    } else {
        collide<typename Form<FORM>::R, COLL, VAR, GM>(v, K);
    }
}

}  // namespace kbc
