// kbc_adjoint.hpp -- reverse-mode derivative (vector-Jacobian product) of the
// per-node collision of kbc_device.hpp.
//
// Given the deviations g of a pre-collision state and the adjoint mu of the
// post-collision deviations, collide_vjp returns lam = J^T mu, J = dg'/dg, and
// the node's contribution mu . dg'/dbeta.  The stabiliser gamma(f) of
// eq. (result21) is by default differentiated with the rest of the collision through
// <ds|dh>, <dh|dh> and the entropic weights 1/feq; where the denominator guard
// selects gamma = 2 it is a constant.  The exact stabiliser (the root of
// eq. (result1), found by iteration) is differentiated by the implicit
// function theorem at the root: for F(gamma; ds, dh, 1/feq, beta) = 0,
// d gamma = -(dF at fixed gamma) / F'(gamma).  The forward quantities of the KBC
// collision come from kbc_forward(), the code collide() runs, so both take the
// same guard decisions on the same values; the chain rule then runs through
// them in reverse order.
#pragma once

#include "kbc_device.hpp"

namespace kbc {

// Sum of one double per lane over the wave, in a fixed order.
__device__ __forceinline__ double wave_sum_d(double v) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// Moment adjoints from the adjoints p of populations in kbc_forward's scaled
// units: of T, N, Pi and of half of Q_xyy, Q_yxx and A.
template <typename R> struct MomAdj {
    R T, N, P, x, y, a;
};
template <typename R>
__device__ __forceinline__ MomAdj<R> moments_adj(const R (&p)[9]) {
    MomAdj<R> m;
    const R a1 = p[1] + p[3], a2 = p[2] + p[4], f57 = p[5] + p[7], f68 = p[6] + p[8];
    const R e57 = p[5] - p[7], e86 = p[8] - p[6];
    const R ax = a1 + a2;
    m.T = fmaR(R(0.25), ax, R(-0.5) * p[0]);
    m.N = R(0.25) * (a1 - a2);
    m.P = R(0.5) * (f57 - f68);
    m.x = (p[3] - p[1]) + (e57 + e86);
    m.y = (p[4] - p[2]) + (e57 - e86);
    m.a = (p[0] - ax) + (f57 + f68);
    return m;
}

// FROZEN = true holds gamma at its forward value (the derivative of the map
// with the stabiliser treated as a per-node constant).
template <typename R, int COLL, int VAR, int GM, bool FROZEN = false>
__device__ __forceinline__ void collide_vjp(const R (&g)[9], const R (&mu)[9], const Coef<R>& K,
                                            R (&lam)[9], R& dbeta) {
    // adjoints of rho - rho0, j and u collected below
    R drb = R(0), jxb = R(0), jyb = R(0), uxb = R(0), uyb = R(0);
    // adjoints of the raw sums of g: sum c_x^2 g, sum c_y^2 g, sum c_x c_y g,
    // sum c_x c_y^2 g, sum c_x^2 c_y g, sum c_x^2 c_y^2 g
    R Sxxb = R(0), Syyb = R(0), Sxyb = R(0), Qxrb = R(0), Qyrb = R(0), Arb = R(0);
    R ir, ux, uy;

    if constexpr (COLL == LBGK) {
        const R s13 = g[1] + g[3], s24 = g[2] + g[4], s57 = g[5] + g[7], s68 = g[6] + g[8];
        const R d13 = g[1] - g[3], d24 = g[2] - g[4], d57 = g[5] - g[7], d68 = g[6] - g[8];
        const R dr = (g[0] + (s57 + s68)) + (s13 + s24);
        const R jx = d13 + (d57 - d68), jy = d24 + (d57 + d68);
        const R rho = K.rho0 + dr;
        ir = rcpR(rho);
        ux = jx * ir;
        uy = jy * ir;
        const R uxx = ux * ux, uyy = uy * uy, u2 = uxx + uyy;
        const R upv = ux + uy, umv = ux - uy;
        // g' = g - 2 beta (g - feqd); feqd_i = W_i [ (rho - rho0) + rho e_i ]
        const R c0 = R(-1.5) * u2;
        const R bx = fmaR(R(4.5), uxx, c0), by = fmaR(R(4.5), uyy, c0);
        const R bp = fmaR(R(4.5) * upv, upv, c0), bm = fmaR(R(4.5) * umv, umv, c0);
        R e[9];
        e[0] = c0;
        e[1] = fmaR(R(3), ux, bx);
        e[3] = fmaR(R(-3), ux, bx);
        e[2] = fmaR(R(3), uy, by);
        e[4] = fmaR(R(-3), uy, by);
        e[5] = fmaR(R(3), upv, bp);
        e[7] = fmaR(R(-3), upv, bp);
        e[8] = fmaR(R(3), umv, bm);
        e[6] = fmaR(R(-3), umv, bm);
        const R tb = R(2) * K.beta;
        R db = R(0);
        // feqd_i depends on dr (directly and through rho) and on u through e_i:
        // d feqd_i / d dr = W_i (1 + e_i), d e_i / d u = 3 c_i + 9 (c_i.u) c_i - 3 u
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            const R feqd = R(weight(i)) * fmaR(rho, e[i], dr);
            db = fmaR(mu[i], g[i] - feqd, db);
            const R fb = tb * mu[i];                 // adjoint of feqd_i
            const R wr = R(weight(i)) * fb;
            drb = fmaR(wr, R(1) + e[i], drb);
            const R cu = R(kCx[i]) * ux + R(kCy[i]) * uy;
            const R eb = wr * rho;                   // adjoint of e_i
            uxb = fmaR(eb, fmaR(R(9) * cu, R(kCx[i]), fmaR(R(-3), ux, R(3) * R(kCx[i]))), uxb);
            uyb = fmaR(eb, fmaR(R(9) * cu, R(kCy[i]), fmaR(R(-3), uy, R(3) * R(kCy[i]))), uyb);
            lam[i] = (R(1) - tb) * mu[i];
        }
        dbeta = R(-2) * db;
    } else {
        KbcNode<R> n;
        kbc_forward<R, VAR, (GM == GEXACT ? GEST : GM)>(g, K, n);
        constexpr bool kCentral = (VAR == VA || VAR == VB), kTrace = (VAR == VA || VAR == VC);
        constexpr R third = R(1.0 / 3.0);
        ir = n.ir;
        ux = n.ux;
        uy = n.uy;
        const bool active = n.active;
        R gam = n.gam, bg = K.beta * gam;
        if constexpr (GM == GEXACT) {
            if (active) gam = exact_gamma<R>(n, K, bg);
        }

        // --------------------------------------------------------- reverse
        // g'_i = g_i - 2 beta s_i - beta gamma h_i; m_i, sb_i and hb_i are
        // adjoints of the scaled populations s_i node_scale(i), h_i node_scale(i)
        R m[9], sb[9], hb[9];
        R mdh = R(0), mds = R(0);
        const R tb = R(2) * K.beta;
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            lam[i] = mu[i];
            m[i] = (i == 0 || i > 4) ? mu[i] * (R(1) / node_scale<R>(i)) : mu[i];
            mdh = fmaR(m[i], n.dh[i], mdh);
            if (VAR != VD || i) mds = fmaR(m[i], n.ds[i], mds);
            sb[i] = -tb * m[i];
            hb[i] = -bg * m[i];
        }
        // d g'_i / d beta = -(2 s_i + gamma h_i), d g'_i / d gamma = -beta h_i
        const R gamb = -K.beta * mdh;
        dbeta = -fmaR(gam, mdh, R(2) * mds);
        if constexpr (GM != GFIX && !FROZEN) {
            R wd[9];                                   // adjoints of the scaled denominators d_i
            if constexpr (GM == GEXACT) {
#pragma unroll
                for (int i = 0; i < 9; ++i) wd[i] = R(0);
                if (active) {
                    // F = sum_i dh_i ln(1 + x_i), x_i = y_i wr_i,
                    // y_i = (1 - beta gamma) dh_i - (2 beta - 1) ds_i, wr_i = w_i / rho:
                    // dF/d dh_i = ln(1 + x_i) + (1 - beta gamma) dh_i wr_i / (1 + x_i),
                    // dF/d ds_i = -(2 beta - 1) dh_i wr_i / (1 + x_i),
                    // dF/d wr_i = dh_i y_i / (1 + x_i),
                    // dF/d beta = -sum_i dh_i (gamma dh_i + 2 ds_i) wr_i / (1 + x_i),
                    // F'(gamma) = -beta sum_i dh_i^2 wr_i / (1 + x_i)
                    R ds[9], dh[9], w[9];
                    unscaled(n, ds, dh, w);
                    const R om = R(1) - bg, tbm1 = R(2) * K.beta - R(1);
                    R wr[9], y[9], r[9], lg[9];
                    R D = R(0);
                    bool ok = true;
#pragma unroll
                    for (int i = 0; i < 9; ++i) {
                        wr[i] = w[i] * ir;
                        y[i] = fmaR(om, dh[i], -(tbm1 * ds[i]));
                        const R x = y[i] * wr[i];
                        ok = ok && (x > R(-1));
                        r[i] = rcpR(R(1) + x);
                        lg[i] = log1pR(x);
                        D = fmaR(-K.beta * dh[i] * dh[i] * wr[i], r[i], D);
                    }
                    // where the iteration stopped short of a root (an argument
                    // of the logarithm left (0, inf), or F' >= 0) gamma is held
                    const R imp = (ok && D < R(0)) ? -gamb / D : R(0);   // -gamma_bar / F'
                    R irb = R(0), fb = R(0);
#pragma unroll
                    for (int i = 0; i < 9; ++i) {
                        const R k = R(1) / node_scale<R>(i), k2 = k * k;
                        const R t = dh[i] * wr[i] * r[i];
                        hb[i] = fmaR(imp * k, fmaR(om, t, lg[i]), hb[i]);
                        sb[i] = fmaR(imp * k, -tbm1 * t, sb[i]);
                        const R wrb = imp * dh[i] * y[i] * r[i];
                        irb = fmaR(wrb, w[i], irb);
                        wd[i] = -(wrb * ir) * w[i] * w[i] * k2;
                        fb = fmaR(t, fmaR(gam, dh[i], R(2) * ds[i]), fb);
                    }
                    dbeta = fmaR(-imp, fb, dbeta);
                    drb = -(irb * ir) * ir;                    // ir = 1 / (rho0 + dr)
                }
            } else {
                // gamma = 1/beta - (2 - 1/beta) a / b with a = sum s h w, b = sum h h w
                // (c enters the guard only); ab, bb: adjoints of a and b, zero where
                // the guard holds gamma at 2
                const R ib2 = K.inv_beta * K.inv_beta;
                const R gb = active ? gamb : R(0);
                const R ratio = active ? n.ratio : R(0);
                dbeta = fmaR(gb, -(R(1) + ratio) * ib2, dbeta);
                const R ab = active ? -K.two_m_inv_beta * gb * rcpR(n.b) : R(0);
                const R bb = -ab * ratio;
#pragma unroll
                for (int i = 0; i < 9; ++i) {
                    // adjoint of w_i = 1 / d_i: h_i (ab s_i + bb h_i)
                    const R hw = n.dh[i] * n.w[i];
                    R q = bb * hw;
                    if (VAR != VD || i) q = fmaR(ab, n.ds[i] * n.w[i], q);
                    sb[i] = fmaR(ab, hw, sb[i]);
                    hb[i] += fmaR(bb, hw, q);
                    wd[i] = -hw * q;
                }
            }
            // d_i in u: a quarter of the rest population's 1/9 - |u|^2 / 6, axes
            // 1/9 - |u|^2 / 6 + u_a^2 / 2 +- u_a / 3, four times the diagonals'
            // 1/9 + |u|^2 / 3 +- u_x u_y + (c.u) / 3
            const R p13 = wd[1] + wd[3], p24 = wd[2] + wd[4], p57 = wd[5] + wd[7], p68 = wd[6] + wd[8];
            const R m57 = wd[5] - wd[7], m86 = wd[8] - wd[6];
            const R pd = p57 + p68, dq = p57 - p68;
            const R cx = fmaR(R(2), p13 + pd, -(p24 + wd[0])), cy = fmaR(R(2), p24 + pd, -(p13 + wd[0]));
            uxb = fmaR(third, fmaR(ux, cx, (wd[1] - wd[3]) + (m57 + m86)), uy * dq);
            uyb = fmaR(third, fmaR(uy, cy, (wd[2] - wd[4]) + (m57 - m86)), ux * dq);
        }
        const MomAdj<R> sm = moments_adj<R>(sb), hm = moments_adj<R>(hb);
        R Tb = kTrace ? sm.T : hm.T, Nb = sm.N, Pb = sm.P;
        if constexpr (kCentral) {
            // h = df - s takes Q and A less the shear part's: ox, oy, a2 (the
            // halves of Q_s, A_s), a2 = u_x ox + u_y oy, ox = u_y Pi + u_x (T_s - N) / 4,
            // oy = u_x Pi + u_y (T_s + N) / 4
            const R a2b = sm.a - hm.a;
            const R oxb = fmaR(ux, a2b, sm.x - hm.x), oyb = fmaR(uy, a2b, sm.y - hm.y);
            Pb = fmaR(uy, oxb, fmaR(ux, oyb, Pb));
            const R tm = ux * oxb, tp = uy * oyb;
            Nb = fmaR(R(0.25), tp - tm, Nb);
            if constexpr (kTrace) Tb = fmaR(R(0.25), tp + tm, Tb);
            uxb = fmaR(a2b, n.ox, fmaR(n.tmn, oxb, fmaR(n.dP, oyb, uxb)));
            uyb = fmaR(a2b, n.oy, fmaR(n.dP, oxb, fmaR(n.tpn, oyb, uyb)));
        }
        Qxrb = R(0.5) * hm.x;
        Qyrb = R(0.5) * hm.y;
        Arb = R(0.5) * hm.a;
        // dT = sum c^2 g - 2/3 dr - rho |u|^2, dN = ... - rho (u_x^2 - u_y^2),
        // dP = ... - rho u_x u_y, dQ_a = ... - j_a / 3, dA = ... - dr / 9 - rho |u|^2 / 3
        const R J = fmaR(third, Arb, Tb);
        const R Cx = J + Nb, Cy = J - Nb;
        jxb = -fmaR(Cx, ux, fmaR(Pb, uy, third * Qxrb));
        jyb = -fmaR(Cy, uy, third * Qyrb);
        uxb = fmaR(-Cx, n.jx, uxb);
        uyb = fmaR(-Cy, n.jy, fmaR(-Pb, n.jx, uyb));
        drb -= fmaR(R(2.0 / 3.0), Tb, R(1.0 / 9.0) * Arb);
        Sxxb = Tb + Nb;
        Syyb = Tb - Nb;
        Sxyb = Pb;
    }
    // u = j / rho, rho = rho0 + dr
    jxb = fmaR(uxb, ir, jxb);
    jyb = fmaR(uyb, ir, jyb);
    drb = fmaR(-ir, fmaR(uxb, ux, uyb * uy), drb);
    // dr = sum g, j = sum c g, and the raw sums of g:
    // lam_i += drb + c_x jxb + c_y jyb + c_x^2 Sxxb + c_y^2 Syyb + c_x c_y Sxyb
    //          + c_x c_y^2 Qxrb + c_x^2 c_y Qyrb + c_x^2 c_y^2 Arb
    const R ax = drb + Sxxb, ay = drb + Syyb;
    const R dd = (ax + Syyb) + Arb;               // common to the diagonals
    const R px = jxb + Qxrb, py = jyb + Qyrb;
    lam[0] += drb;
    lam[1] += ax + jxb;
    lam[3] += ax - jxb;
    lam[2] += ay + jyb;
    lam[4] += ay - jyb;
    const R dp = dd + Sxyb, dm = dd - Sxyb;
    lam[5] += dp + (px + py);
    lam[7] += dp - (px + py);
    lam[6] += dm - (px - py);
    lam[8] += dm + (px - py);
}

}  // namespace kbc
