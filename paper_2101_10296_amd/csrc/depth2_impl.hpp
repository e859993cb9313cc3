// Depth p = 2 on trees: <Z_u Z_v> and its derivatives in closed form.
//
// Where every qubit at distance 1 couples to one of u and v alone and every qubit at distance 2 to
// one of those alone, the qubits off the edge are traced out one by one.  A neighbour a of u
// (coupling w) sees u's bit on four occasions: before and behind layer 1, in psi and its
// conjugate.  With t_l = gamma_l delta, f = prod over its leaves of cos(t_1 x) (shell.hpp), its trace is
//   1, alpha -+ i sb f X, kappa, kappa alpha -+ cb X    (alpha = cos t_2 w, kappa = cos t_1 w,
//   X = sin t_1 w sin t_2 w; cb, sb = cos, sin of 2 beta_1)
// as u's bit differs between psi and its conjugate nowhere, behind, before, or on both sides of layer
// 1; the sign is that of u's bit behind against before.  Products over a side's neighbours:
//   g = prod (alpha - i sb f X), k = prod kappa, h+- = prod (kappa alpha -+ cb X),
//   H1 = (h+ - h-) / 2 + cb (h+ + h-) / 2, H2 = (h+ + h-) / 2 + cb (h+ - h-) / 2.
// The sum over the edge's own bits, with p_l = t_l w_uv and C, S = cos, sin of 2 beta_2, is
//   <ZZ> = -sin p_1 T1 - sin p_2 T2,
//   T1 = C^2 cb sb (k_u + k_v) + C S cos p_2 (cb (H1_u + H1_v) - sb^2 (Re g_u k_v + Re g_v k_u))
//        - S^2 sb (Re g_u H1_v + Re g_v H1_u),
//   T2 = C S (cos p_1 (H2_u + H2_v) - sb (Im g_u + Im g_v)).
// The products carry their derivatives along; all in FP64, some 50 operations a neighbour.
#pragma once

#include "depth2.hpp"

namespace qaoa {

// One neighbour's cosines, sines and their derivatives in t_1 and t_2.
struct D2Val {
    double ka, al, s1, s2;         // cos t_1 w, cos t_2 w, sin t_1 w, sin t_2 w
    double w, f, f1;               // its leaves' f and df/dt_1
};

__device__ __forceinline__ D2Val d2_val(const D2Type& t, const D2Leaf* leaf, double t1, double t2) {
#pragma clang fp contract(off)
    D2Val v;
    v.w = t.w;
    sincos(t1 * t.w, &v.s1, &v.ka);
    sincos(t2 * t.w, &v.s2, &v.al);
    v.f = 1.0;
    v.f1 = 0.0;
    for (int i = 0; i < t.n_leaf; ++i) {
        const D2Leaf L = leaf[t.leaf + i];
        double s, c;
        sincos(t1 * L.w, &s, &c);
        for (int j = 0; j < L.m; ++j) {
            v.f1 = fma(v.f1, c, -(v.f * (L.w * s)));
            v.f *= c;
        }
    }
    return v;
}

struct D2Angles {
    double cb, sb, C, S;
};

// Products over one side's neighbours; [0..2]: derivatives in t_1, t_2, beta_1.
template <bool GRAD>
struct D2Side {
    double gr, gi, k, H1, H2;
    double gr_[GRAD ? 3 : 1], gi_[GRAD ? 3 : 1], k_, H1_[GRAD ? 3 : 1], H2_[GRAD ? 3 : 1];
};

template <bool GRAD, class Get>
__device__ __forceinline__ D2Side<GRAD> d2_side(int n, const D2Angles& a, const Get& get) {
#pragma clang fp contract(off)
    double gr = 1.0, gi = 0.0, k = 1.0, hp = 1.0, hm = 1.0;
    double gr_[3] = {}, gi_[3] = {}, k_ = 0.0, hp_[3] = {}, hm_[3] = {};
    for (int i = 0; i < n; ++i) {
        const D2Val v = get(i);
        const double X = v.s1 * v.s2, y = -a.sb * (v.f * X), ka = v.ka * v.al;
        const double Fp = fma(-a.cb, X, ka), Fm = fma(a.cb, X, ka);
        if constexpr (GRAD) {
            const double ka1 = -v.w * v.s1, al2 = -v.w * v.s2, X1 = v.w * (v.ka * v.s2), X2 = v.w * (v.s1 * v.al);
            // factor of g: al + i y, and its derivatives d + i y_
            const double y_[3] = {-a.sb * fma(v.f1, X, v.f * X1), -a.sb * (v.f * X2), -2.0 * a.cb * (v.f * X)};
            const double kal[2] = {ka1 * v.al, v.ka * al2};
            const double Xd[2] = {X1, X2};
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                double r = fma(gr_[d], v.al, -(gi_[d] * y)), m = fma(gr_[d], y, gi_[d] * v.al);
                r = fma(-gi, y_[d], r);
                m = fma(gr, y_[d], m);
                if (d == 1) {
                    r = fma(gr, al2, r);
                    m = fma(gi, al2, m);
                }
                gr_[d] = r;
                gi_[d] = m;
                const double p = d < 2 ? fma(-a.cb, Xd[d], kal[d]) : 2.0 * a.sb * X;
                const double q = d < 2 ? fma(a.cb, Xd[d], kal[d]) : -2.0 * a.sb * X;
                hp_[d] = fma(hp_[d], Fp, hp * p);
                hm_[d] = fma(hm_[d], Fm, hm * q);
            }
            k_ = fma(k_, v.ka, k * ka1);
        }
        const double r = fma(gr, v.al, -(gi * y));
        gi = fma(gr, y, gi * v.al);
        gr = r;
        k *= v.ka;
        hp *= Fp;
        hm *= Fm;
    }
    D2Side<GRAD> s;
    s.gr = gr;
    s.gi = gi;
    s.k = k;
    const double hs = 0.5 * (hp + hm), hd = 0.5 * (hp - hm);
    s.H1 = fma(a.cb, hs, hd);
    s.H2 = fma(a.cb, hd, hs);
    if constexpr (GRAD) {
        s.k_ = k_;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const double ps = 0.5 * (hp_[d] + hm_[d]), pd = 0.5 * (hp_[d] - hm_[d]);
            s.gr_[d] = gr_[d];
            s.gi_[d] = gi_[d];
            s.H1_[d] = fma(a.cb, ps, pd);
            s.H2_[d] = fma(a.cb, pd, ps);
            if (d == 2) {
                s.H1_[d] = fma(-2.0 * a.sb, hs, s.H1_[d]);
                s.H2_[d] = fma(-2.0 * a.sb, hd, s.H2_[d]);
            }
        }
    }
    return s;
}

// v[0]: <ZZ>; GRAD: v[1..4]: its derivatives in t_1, t_2, beta_1, beta_2.  e: the edge; u, w: its sides.
template <bool GRAD>
__device__ __forceinline__ void d2_term(const D2Val& e, const D2Side<GRAD>& u, const D2Side<GRAD>& w, const D2Angles& a,
                                        double (&v)[5]) {
#pragma clang fp contract(off)
    const double cb = a.cb, sb = a.sb, C = a.C, S = a.S, CS = C * S, sb2 = sb * sb, cs = cb * sb;
    const double K = u.k + w.k, H = u.H1 + w.H1, Q = fma(u.gr, w.k, w.gr * u.k), R = fma(u.gr, w.H1, w.gr * u.H1);
    const double H2 = u.H2 + w.H2, G = u.gi + w.gi;
    const double B = fma(cb, H, -(sb2 * Q)), D = fma(e.ka, H2, -(sb * G));
    const double T1 = fma(C * C, cs * K, fma(CS, e.al * B, -(S * S * (sb * R))));
    const double T2 = CS * D;
    v[0] = -fma(e.s1, T1, e.s2 * T2);
    if constexpr (GRAD) {
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const double ku = d == 0 ? u.k_ : 0.0, kw = d == 0 ? w.k_ : 0.0;
            const double Hd = u.H1_[d] + w.H1_[d], H2d = u.H2_[d] + w.H2_[d], Gd = u.gi_[d] + w.gi_[d];
            double Qd = fma(u.gr_[d], w.k, w.gr_[d] * u.k);
            if (d == 0) Qd = fma(u.gr, kw, fma(w.gr, ku, Qd));
            const double Rd = fma(u.gr_[d], w.H1, fma(w.gr_[d], u.H1, fma(u.gr, w.H1_[d], w.gr * u.H1_[d])));
            double Bd = fma(cb, Hd, -(sb2 * Qd)), Dd = fma(e.ka, H2d, -(sb * Gd)), K1 = d == 0 ? cs * (ku + kw) : 0.0;
            double Rs = sb * Rd, x = 0.0;
            if (d == 0) x = e.w * (e.ka * T1 - e.s2 * (CS * (e.s1 * H2)));
            if (d == 1) x = e.w * (e.al * T2 - e.s1 * (CS * (e.s2 * B)));
            if (d == 2) {   // cb, sb outside the sides
                Bd = fma(-2.0 * sb, H, fma(-4.0 * cs, Q, Bd));
                Dd = fma(-2.0 * cb, G, Dd);
                K1 = 2.0 * fma(cb, cb, -sb2) * K;
                Rs = fma(2.0 * cb, R, Rs);
            }
            const double T1d = fma(C * C, K1, fma(CS, e.al * Bd, -(S * S * Rs)));
            v[1 + d] = -(fma(e.s1, T1d, e.s2 * (CS * Dd)) + x);
        }
        const double c2 = fma(C, C, -(S * S));   // d(CS) = 2 c2, d(C^2) = -4 CS, d(S^2) = 4 CS
        const double T1b = fma(-4.0 * CS, cs * K, fma(2.0 * c2, e.al * B, -(4.0 * CS * (sb * R))));
        v[4] = -fma(e.s1, T1b, e.s2 * (2.0 * c2 * D));
    }
}

__device__ __forceinline__ D2Angles d2_angles(double b1, double b2) {
    D2Angles a;
    sincos(2.0 * b1, &a.sb, &a.cb);
    sincos(2.0 * b2, &a.S, &a.C);
    return a;
}

// One cone from its types.
template <bool GRAD>
__device__ __forceinline__ void d2_cone(const D2Args& a, const D2Cone& c, double t1, double t2, const D2Angles& an,
                                        double (&v)[5]) {
    auto val = [&](int t) { return d2_val(a.types[t], a.leaf, t1, t2); };
    auto side = [&](int q) {
        const D2SideDef d = a.sides[q];
        return d2_side<GRAD>(d.n, an, [&](int i) { return val(a.branch[d.off + i]); });
    };
    d2_term<GRAD>(val(c.edge), side(c.u), side(c.v), an, v);
}

}  // namespace qaoa
