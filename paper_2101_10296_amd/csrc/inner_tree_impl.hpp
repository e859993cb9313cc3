// Light cones at depth 2 whose shell qubits are leaves, each next to one inner qubit: one 16-lane row
// per cone.
//
// With the leaves dephased (shell.hpp) a cone of a 3-regular graph is 2^4 choices of signs on its
// 6 inner qubits, 6 of them up to the cone's symmetries, in place of 81 configurations of the
// leaves (41 up to the flip, 12 listed).  No configuration of the shell is left that a flip of
// every qubit could change, so each state has the symmetry psi(~x) = s psi(x), s = (-1)^(signs):
// the last inner qubit is dropped, and its X flips the others, times s.  That leaves eight states
// of 2^5 amplitudes for a row (two lanes each), four cones for a wave, where a wave ran the 16
// states of 2^6 amplitudes of one cone.  Layout, gauge and last layer are those of inner_impl.hpp;
// the dropped qubit pairs register r with A - 1 - r, over the lane qubit (7 vs 4 instructions per
// four amplitudes, as a pair cannot be turned in place).
//
// Bound: vector instruction issue (about 1100 instructions of a wave per round of its four cones).
// Measured on one MI355X, energy and gradient at p = 2 of random 3-regular graphs: n = 10000, 256
// points, 215.6 ms on the kernels for whole cones, 7.49 ms a wave per cone, 2.32 ms here; seven
// graphs of 6000 to 375 nodes, 8 points, 10.6 ms, 429 us, 188 us; n = 1000, 64 points, with the
// training step around it, 5.35 ms, 253 us, 146-180 us (host).
#pragma once

#include "inner_impl.hpp"

namespace qaoa {

// a[i] += flip(b[3 - i]) t and back, flip: lane xor 1
__device__ __forceinline__ void row_cross2(float2& a, float2& b, float2& c, float2& d, float t) {
    float2 x, y;
    asm volatile("s_nop 1\n"
                 "v_mov_b32 %8, %0\n"
                 "v_mov_b32 %9, %1\n"
                 "v_mov_b32 %10, %2\n"
                 "v_mov_b32 %11, %3\n"
                 "v_fmac_f32_dpp %0, %6, %12 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n"
                 "v_fmac_f32_dpp %1, %7, %12 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n"
                 "v_fmac_f32_dpp %2, %4, %12 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n"
                 "v_fmac_f32_dpp %3, %5, %12 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n"
                 "v_fmac_f32_dpp %4, %10, %12 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n"
                 "v_fmac_f32_dpp %5, %11, %12 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n"
                 "v_fmac_f32_dpp %6, %8, %12 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n"
                 "v_fmac_f32_dpp %7, %9, %12 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf"
                 : "+v"(a.x), "+v"(a.y), "+v"(b.x), "+v"(b.y), "+v"(c.x), "+v"(c.y), "+v"(d.x), "+v"(d.y), "=&v"(x.x),
                   "=&v"(x.y), "=&v"(y.x), "=&v"(y.y)
                 : "v"(t));
}

// The dropped qubit's mixer 1 - i t X (t with the state's s).
template <int KIN, int A>
__device__ __forceinline__ void tr_mix(float2 (&v)[A], float t, const float (&sg)[4]) {
    if constexpr (Iz<KIN - 1>::LB == 1) {
        const float ts = t * sg[0];
#pragma unroll
        for (int r = 0; r < A / 2; r += 2) row_cross2(v[r], v[r + 1], v[A - 2 - r], v[A - 1 - r], ts);
    } else {
#pragma unroll
        for (int r = 0; r < A / 2; ++r) {
            bfly(v[r], v[A - 1 - r], t);
            if ((r & 3) == 3) __builtin_amdgcn_sched_barrier(0);
        }
    }
}

// Im <l| X |f> of the dropped qubit, this lane's share, without s.
template <int KIN, int A>
__device__ __forceinline__ float tr_xsum(const float2 (&f)[A], const float2 (&l)[A], const float (&sg)[4]) {
    float a0 = 0.f, a1 = 0.f;
    if constexpr (Iz<KIN - 1>::LB == 1) {
        float2 x[A];
#pragma unroll
        for (int r = 0; r < A; ++r) x[r] = f[A - 1 - r];
#pragma unroll
        for (int r = 0; r < A; r += 4) row_dot4<0>(a0, a1, x, l, r);
        return sg[0] * (a0 + a1);
    } else {
#pragma unroll
        for (int r = 0; r < A / 2; r += 2) {
            const int s = A - 1 - r;
            xacc2(a0, a1, l[r], l[s], f[r], f[s], l[r + 1], l[s - 1], f[r + 1], f[s - 1]);
        }
        return a0 + a1;
    }
}

// Sum over a row, the same in every lane.
__device__ __forceinline__ double row_sum(double x) {
    static_for<0, 4>([&](auto I) {
        constexpr int i = decltype(I)::value;
        const long long b = __double_as_longlong(x);
        const float lo = row_flip<i>(__int_as_float(static_cast<int>(b)));
        const float hi = row_flip<i>(__int_as_float(static_cast<int>(b >> 32)));
        const long long o = (static_cast<long long>(__float_as_int(hi)) << 32) |
                            static_cast<long long>(static_cast<unsigned>(__float_as_int(lo)));
        x += __longlong_as_double(o);
    });
    return x;
}

// f and its derivative of every choice of leaves in the plan, from the cosines of in_rows (a barrier
// before, one behind).
__device__ __forceinline__ void tr_types(const InArgs& a, int tid, int threads, const float2* dyn, double2* typ) {
    for (int i = tid; i < a.n_types; i += threads) typ[i] = z_factor(a.types[i], reinterpret_cast<const double2*>(dyn));
}

// Cone c by one row, where live: put(code, value) as in in_unit.
template <int KIN, bool GRAD, class Put>
__device__ __forceinline__ void tr_row(const InArgs& a, const ConeTr* cone, bool live, int lane, const InLane<KIN - 1>& ln,
                                       const float2* dyn0, const double2* typ, const InShared& sh, const Put& put) {
    using H = Iz<KIN - 1>;
    constexpr int A = H::A, SLOTS = 16 >> H::LB;
    const int R = a.R;
    const float2* dyn = in_phase(a, const_cast<float2*>(dyn0));
    const ConeTr cd = *cone;
    const float cs2 = static_cast<float>(sh.cs[0] * sh.cs[1]), ss2 = static_cast<float>(sh.cs[1] * sh.cs[1]);
    const uint32_t xl = ln.xl;
    Tab<A> T;
    T.load(a.tab + static_cast<size_t>(cd.tab_off) * 16 + (xl << H::RB));
    const int n_cfg = live ? cd.n_cfg : 0;
    const double C = sh.cs[0], S = sh.cs[1];
    const float t1 = sh.t[1];
    double Zs = 0.0, Bs = 0.0, Gp = 0.0, B1 = 0.0, G1 = 0.0;
    for (int c = (lane & 15) >> H::LB; __any(c < n_cfg); c += SLOTS) {
        const uint32_t e = c < n_cfg ? a.trcfg[cd.cfg_off + c] : 0u;
        double wt = static_cast<double>(e >> 8), dwt = 0.0;
        uint32_t ty = cd.types;
#pragma unroll
        for (int q = 2; q < KIN; ++q, ty >>= 8) {
            const double2 f = typ[ty & 255u];
            const double s = (e >> q) & 1u ? -0.5 : 0.5;
            const double v = fma(s, f.x, 0.5);
            dwt = dwt * v + wt * (s * f.y);
            wt *= v;
        }
        const float sz = __builtin_popcount(e & 255u) & 1 ? -1.f : 1.f;
        // row index of table value 0 in layer 1: the signs are two steps of the gauge
        const uint32_t g0 = ln.gz + 2u * static_cast<uint32_t>(__builtin_popcount((e >> H::RB) & xl));
        const uint32_t s2 = KIN > 3 ? (e >> 1) & 2u : 0u, s3 = KIN > 4 ? (e >> 2) & 2u : 0u;
        int cb[4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
            cb[i] = cd.base + static_cast<int>((g0 + (i & 1 ? s2 : 0u) + (i & 2 ? s3 : 0u)) & 3u) * R;
        float2 f[A];
#pragma unroll
        for (int q = 0; q < A; ++q) f[q] = dyn[T.at(q) + cb[q >> 2]];
        __builtin_amdgcn_sched_barrier(0);
        in_mix<KIN - 1, true>(f, t1, KIN - 1, ln.sg);
        tr_mix<KIN>(f, t1 * sz, ln.sg);
        T.opaque();
        float2 l[GRAD ? A : 1];
        double zv = 0.0, iv = 0.0, dv = 0.0;
        float gp = 0.f;
        in_last<GRAD>(f, l, T, dyn + 4 * R + cd.base, static_cast<float>(cd.base) - cd.mid, cs2, ss2, zv, iv, dv, gp);
        const double E = zv + 2.0 * C * S * iv + S * S * dv;
        Zs = fma(wt, E, Zs);
        if constexpr (GRAD) {
            Bs = fma(wt, 2.0 * (2.0 * (C * C - S * S) * iv + 2.0 * C * S * dv), Bs);
            Gp = fma(wt, static_cast<double>(gp), Gp);
            float b1 = in_xsum<KIN - 1, true>(f, l, KIN - 1, ln.sg);
            b1 = fmaf(sz, tr_xsum<KIN>(f, l, ln.sg), b1);
            B1 = fma(wt, static_cast<double>(b1), B1);
            in_mix<KIN - 1, true>(l, -t1, KIN - 1, ln.sg);
            tr_mix<KIN>(l, -t1 * sz, ln.sg);
            float g1 = 0.f;
            T.opaque();
            const float cm = static_cast<float>(cd.base) - cd.mid;
#pragma unroll
            for (int q = 0; q < A; ++q) {
                const float2 t = dyn[T.at(q) + cb[q >> 2]];
                const float im = fmaf(l[q].x, t.y, -l[q].y * t.x);
                g1 = fmaf(static_cast<float>(T.at(q)) + cm, im, g1);
                if ((q & 7) == 7) __builtin_amdgcn_sched_barrier(0);
            }
            G1 = fma(wt, 2.0 * static_cast<double>(g1), fma(dwt, E, G1));
        }
    }
    // |psi|^2 carries 2^kin (generation without its norm) and 1 / |kappa_1|^(2 kin), and the sums run
    // over half of the amplitudes
    double k = sh.k2[1], k1 = 1.0;
#pragma unroll
    for (int e = KIN; e; e >>= 1) {
        if (e & 1) k1 *= k;
        k *= k;
    }
    const double nz = exp2(1.0 - static_cast<double>(KIN)) * k1;
    if constexpr (GRAD) {
        double v[8] = {nz * Zs, nz * Bs, 2.0 * nz * Gp, 2.0 * nz * B1, nz * G1, 0.0, 0.0, 0.0};
        const double x = lane_sum8<false>(v, lane);
        const int i = (lane & 8 ? 4 : 0) | (lane & 3);   // the value that this lane holds
        if (live && !(lane & 4) && i < 5) put(cd.orbit, i == 0 ? 0 : i == 1 ? 4 : i == 2 ? 2 : i == 3 ? 3 : 1, x);
    } else {
        const double x = row_sum(nz * Zs);
        if (live && (lane & 15) == 0) put(cd.orbit, 0, x);
    }
}

}  // namespace qaoa
