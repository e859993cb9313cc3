// Light cones on 11 to 14 inner qubits, one workgroup per unit of work (p = 2, 3).
//
// The same reduction as inner_impl.hpp where the inner state exceeds a wave: 16 amplitudes per
// thread in the two layouts of whole_impl.hpp (L0: qubits 0-3 in registers, 4-7 on the lanes of a
// row; L1: the qubits above in registers and row lanes), every qubit in the gauge i^|x|.  Only
// layer 1 mixes more than eight qubits, so psi goes through LDS once (L1 -> L0) and lambda once
// on its way back; all other layers stay in registers and rows.  In the gauge the last layer's
// cos Z + sin Y (of 2 beta_p) is the real cos Z - sin X.  The beta_1 terms of the upper qubits
// are taken at the start of layer 1 with D_1 |+> made again, those of qubits 0-7 behind it.
//
// A 30-qubit cone of a 3-regular graph at p = 3 has 14 inner qubits and a shell of 16 leaves: 256
// choices of signs, 21 up to the cone's symmetries, of 2^14 amplitudes that never leave the compute
// unit, in place of seven sweeps over 2^29 amplitudes in device memory.  90 terms of 19 to 30
// qubits, energy and gradient: 257 -> 20.5 ms with listed configurations of the leaves, 8.9 with
// lists up to any symmetry, 7.0 with signs (5.5 of it in the passes of cones of up to 24 qubits).
// Bound: vector instruction issue (about 200 per amplitude with the gradient) at one to two
// workgroups per CU (LDS).
#pragma once

#include "whole_impl.hpp"
#include "wide.hpp"

namespace qaoa {

template <int KIN>
struct Uz {
    static constexpr int KL = KIN;
    static constexpr int RB = 4, A = 16, ROW = 4;
    static constexpr int TB = KIN - RB;
    static constexpr int W = 1 << TB;                         // threads
    static constexpr int REST = TB - ROW;
    static constexpr int NR = REST < RB ? REST : RB;
    static constexpr int NQ = REST - NR;
    static constexpr int reg(int lay, int i) { return lay == 1 && i < NR ? RB + ROW + i : i; }
    static constexpr int row(int lay, int i) { return lay == 1 && i < NQ ? RB + ROW + NR + i : RB + i; }
    static constexpr int up(int lay, int i) { return lay == 0 ? RB + ROW + i : (i < NR ? i : RB + i - NR); }
    // as Wz: the qubits that L1 puts on row lanes take over the weights of those they displace
    static constexpr uint32_t wt(int j) {
        uint32_t w = (1u << j) + ((1u << j) >> 4);
        if (j >= RB + ROW + NR) w += ((16u << (j - RB - ROW - NR)) + (1u << (j - RB - ROW - NR))) & 15u;
        return w;
    }
    static constexpr uint32_t PALL = [] {
        uint32_t s = 0;
        for (int j = 0; j < KL; ++j) s += wt(j);
        return s;
    }();
    static constexpr uint32_t NPAD = PALL + 1;
};

template <class Z, int FROM, int TO, int A>
__device__ __forceinline__ void wtrans(float2 (&v)[A], float2* xb, uint32_t of, uint32_t ot) {
    __syncthreads();
#pragma unroll
    for (int r = 0; r < A; ++r) xb[of + wregp<Z, FROM>(r)] = v[r];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < A; ++r) v[r] = xb[ot + wregp<Z, TO>(r)];
}

// Mixer of the first m <= 8 qubits in L0.
template <int A>
__device__ __forceinline__ void pmix(float2 (&v)[A], float t, int m, const float (&sg)[4]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if (i >= 2 && i >= m) continue;
#pragma unroll
        for (int r = 0; r < A; ++r)
            if (!(r & (1 << i))) rot(v[r], v[r | (1 << i)], t);
        __builtin_amdgcn_sched_barrier(0);
    }
    static_for<0, 4>([&](auto I) {
        constexpr int i = decltype(I)::value;
        if (4 + i < m) {
            const float ts = t * sg[i];
#pragma unroll
            for (int r = 0; r < A; r += 4) row_rot4<i>(v[r], v[r + 1], v[r + 2], v[r + 3], ts);
        }
    });
}

// One register pair of <l|X|f> in the gauge, two pairs per block (see xacc2).
__device__ __forceinline__ void rdot2(float& a0, float& a1, float2 la, float2 lb, float2 pa, float2 pb, float2 lc,
                                      float2 ld, float2 pc, float2 pd) {
    asm volatile("v_fmac_f32 %0, %4, %6\n"
                 "v_fmac_f32 %1, %12, %14\n"
                 "v_fmac_f32 %0, %5, %7\n"
                 "v_fmac_f32 %1, %13, %15\n"
                 "v_fma_f32 %0, -%2, %8, %0\n"
                 "v_fma_f32 %1, -%10, %16, %1\n"
                 "v_fma_f32 %0, -%3, %9, %0\n"
                 "v_fma_f32 %1, -%11, %17, %1"
                 : "+v"(a0), "+v"(a1)
                 : "v"(la.x), "v"(la.y), "v"(lb.x), "v"(lb.y), "v"(pa.x), "v"(pa.y), "v"(pb.x), "v"(pb.y), "v"(lc.x),
                   "v"(lc.y), "v"(ld.x), "v"(ld.y), "v"(pc.x), "v"(pc.y), "v"(pd.x), "v"(pd.y));
}
template <int A>
__device__ __forceinline__ float rdot_bit(int i, const float2 (&f)[A], const float2 (&l)[A]) {
    float a0 = 0.f, a1 = 0.f;
    const int o = i == 0 ? 2 : 1;
#pragma unroll
    for (int r = 0; r < A; ++r)
        if (!(r & ((1 << i) | o))) {
            const int s = r | (1 << i), r2 = r | o, s2 = s | o;
            rdot2(a0, a1, l[r], l[s], f[r], f[s], l[r2], l[s2], f[r2], f[s2]);
        }
    return a0 + a1;
}

// Im <l| sum X_j |f> over the first m <= 8 qubits in L0: over those in registers, and over those of the row
// (FP32 over four qubits each; the two are added in FP64).
template <int A>
__device__ __forceinline__ float2 pxsum(const float2 (&f)[A], const float2 (&l)[A], int m, const float (&sg)[4]) {
    float acc = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i)
        if (i < 2 || i < m) acc += rdot_bit(i, f, l);
    const float regs = acc;
    acc = 0.f;
    static_for<0, 4>([&](auto I) {
        constexpr int i = decltype(I)::value;
        if (4 + i < m) {
            float a0 = 0.f, a1 = 0.f;
#pragma unroll
            for (int r = 0; r < A; r += 4) row_dot4<i>(a0, a1, f, l, r);
            acc = fmaf(sg[i], a0 + a1, acc);
        }
    });
    return make_float2(regs, acc);
}

template <int KIN, bool GRAD, int PP>
__global__ void __launch_bounds__((Uz<KIN>::W), Uz<KIN>::W > 512 ? 4 : 3) k_wide(WdArgs a) {
    using Z = Uz<KIN>;
    constexpr int A = 16, NWV = Z::W / 64;
    __shared__ __attribute__((aligned(16))) float2 xb[Z::NPAD];
    __shared__ CfgWd s_cfg[WD_CFG];
    __shared__ float s_t[4];
    __shared__ double s_k2[4], s_cs[2];
    __shared__ double2 s_z[16];
    __shared__ double s_sum[NWV][8];
    extern __shared__ __attribute__((aligned(16))) float2 dyn0[];   // cosines of the leaves' couplings; phase rows: layer 1 in four gauges, then layers 2..p
    const int tid = threadIdx.x, lane = tid & 63;
    const int R = a.R;
    double2* ct = reinterpret_cast<double2*>(dyn0);
    float2* dyn = dyn0 + 2 * (a.wz + 1);
    const int pt = blockIdx.x / a.n_units, un = blockIdx.x - pt * a.n_units;
    const int point = pt + a.point0;
    const UnitWd unit = a.units[un];
    const ConeWd& cd = a.cones[unit.cone];
    const size_t ip = (static_cast<size_t>(cd.inst) * a.gamma_P + point) * PP;
    const double delta = a.deltas[cd.inst];
    const int n_rows = cd.n_rows;
    for (int i = tid; i < PP * n_rows; i += Z::W) {
        const int l = i / n_rows, j = i - l * n_rows;
        double s, c;
        sincos(a.gamma[ip + l] * delta * static_cast<double>(cd.cut_min + j), &s, &c);
        const float x = static_cast<float>(c), y = static_cast<float>(-s);
        if (l == 0) {   // times 1, i, -1, -i
            dyn[j] = make_float2(x, y);
            dyn[R + j] = make_float2(-y, x);
            dyn[2 * R + j] = make_float2(-x, -y);
            dyn[3 * R + j] = make_float2(y, -x);
        } else {
            dyn[(3 + l) * R + j] = make_float2(x, y);
        }
    }
    for (int j = tid; j <= a.wz; j += Z::W)
        sincos(a.gamma[ip] * delta * static_cast<double>(j), &ct[j].y, &ct[j].x);
    if (tid < PP) {
        double s, c, t, k2;
        sincos(a.beta[ip + tid], &s, &c);
        if (fabs(c) >= fabs(s)) {
            t = s / c;
            k2 = c * c;
        } else {
            t = -c / s;
            k2 = s * s;
        }
        s_t[tid + 1] = static_cast<float>(t);
        s_k2[tid + 1] = k2;
        if (tid == PP - 1) {
            s_cs[0] = c * c - s * s;
            s_cs[1] = 2.0 * s * c;
        }
    }
    __syncthreads();
    // the unit's configurations and their weights (the first wave)
    z_factors(cd.zmask, a.leaf, cd.z_off, ct, tid, s_z);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if (tid < WD_CFG) {
        CfgWd e{};
        const uint32_t c = unit.c0 + tid;
        if (c < unit.c1 && cd.cfg_off >= 0) {
            e = a.cfg[cd.cfg_off + c];
        } else if (c < unit.c1) {   // mixed radix digits (how many of each group's qubits are 1), then signs
            const uint32_t nh = (cd.nc + 1) / 2;
            uint32_t zz = c / nh, rem = c - zz * nh;
            int h[12] = {};
            e.w = ((cd.nc & 1u) && rem == nh - 1) ? 1.0 : 2.0;
            for (uint32_t m = cd.zmask; m; m &= m - 1, zz >>= 1) e.z |= (zz & 1u) << __builtin_ctz(m);
            for (int q = 0; q < cd.n_grp; ++q) {
                const GrpWd& G = a.grp[cd.grp_off + q];
                const uint32_t d = static_cast<uint32_t>(G.m) + 1u;
                const uint32_t nx = rem / d;
                const int t = static_cast<int>(rem - nx * d);
                rem = nx;
                e.c0 += t * G.wsum;
#pragma unroll
                for (int i = 0; i < 12; ++i) h[i] += (G.m - 2 * t) * G.h[i];
                e.w *= kBinom[G.m * 30 + t];
            }
#pragma unroll
            for (int i = 0; i < 12; ++i) e.h[i] = static_cast<int16_t>(h[i]);
        }
        e.dw = z_weight(cd.zmask, e.z, s_z, e.w);
        s_cfg[tid] = e;
    }
    const WhThread th = wh_thread<Z>(static_cast<uint32_t>(tid));
    float sg[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) sg[i] = th.xq[i] ? 1.f : -1.f;
    const uint32_t y0 = wh_base<Z, 0, false>(th), y1 = wh_base<Z, 1, false>(th);
    const uint32_t o0 = wh_base<Z, 0, true>(th), o1 = wh_base<Z, 1, true>(th);
    const int pc = __builtin_popcount(y0);
    const uint8_t* tab = a.tab + cd.tab_off;
    // table bytes: layer 2's (layer 1's inner couplings) in L1, layers 2 .. p in L0
    uint32_t k1[A / 4];
#pragma unroll
    for (int w = 0; w < A / 4; ++w) k1[w] = 0u;
#pragma unroll
    for (int r = 0; r < A; ++r) k1[r >> 2] |= static_cast<uint32_t>(tab[y1 + wreg<Z, 1>(r)]) << (8 * (r & 3));
    auto T1 = [&](int r) { return (k1[r >> 2] >> (8 * (r & 3))) & 255u; };
    Tab<A> T[PP - 1];
#pragma unroll
    for (int l = 0; l < PP - 1; ++l) T[l].load(tab + (static_cast<size_t>(l) << KIN) + y0);
    __syncthreads();
    auto kpow = [&](int l) {   // |kappa_l|^(2 m_l)
        double k = s_k2[l], x = 1.0;
        for (int e = cd.mixed[l]; e; e >>= 1) {
            if (e & 1) x *= k;
            k *= k;
        }
        return x;
    };
    const double k2_1 = kpow(1);
    const float mu1 = static_cast<float>(sqrt(k2_1));
    const float cs2 = static_cast<float>(s_cs[0] * s_cs[1]), ss2 = static_cast<float>(s_cs[1] * s_cs[1]);
    double Zs = 0.0, Is = 0.0, Ds = 0.0, Gp = 0.0, B1 = 0.0, B1u = 0.0, G1 = 0.0, Wd = 0.0;
    double B2 = 0.0, G2 = 0.0;   // PP = 3

    for (uint32_t ci = 0; ci < unit.c1 - unit.c0; ++ci) {
        const CfgWd& e = s_cfg[ci];
        const double wt = e.w;
        // layer-1 row index of this thread's amplitudes in L1: lb + T1 + ca (register bits 0, 1) + cb (2, 3)
        int lb = e.c0 + cd.base[1];
#pragma unroll
        for (int i = 0; i < 4; ++i) lb += th.xq[i] ? e.h[Z::row(1, i) - 2] : 0;
#pragma unroll
        for (int i = 0; i < Z::REST; ++i)
            if (Z::up(1, i) >= 2) lb += ((th.up >> i) & 1u) ? e.h[Z::up(1, i) - 2] : 0;
        auto hr = [&](int i) { return Z::reg(1, i) >= 2 ? static_cast<int>(e.h[Z::reg(1, i) - 2]) : 0; };
        int ca[4], cb[4];
        ca[0] = lb;
        ca[1] = lb + hr(0);
        ca[2] = lb + hr(1);
        ca[3] = ca[1] + hr(1);
        cb[0] = 0;
        cb[1] = hr(2);
        cb[2] = hr(3);
        cb[3] = cb[1] + cb[2];
        // signs: of the thread's qubits two steps of the gauge, of the register qubits a factor
        const uint32_t z = __builtin_amdgcn_readfirstlane(e.z);
        const int pz = pc + 2 * __builtin_popcount(z & y1);
        auto gen = [&](int r) {   // D_1 |+>, gauged, without its norm
            const float2 t = dyn[((pz + __builtin_popcount(r)) & 3) * R + static_cast<int>(T1(r)) + ca[r & 3] + cb[r >> 2]];
            const float x = __builtin_popcount(z & wreg<Z, 1>(r)) & 1 ? -1.f : 1.f;
            return make_float2(x * t.x, x * t.y);
        };
        float2 f[A];
#pragma unroll
        for (int r = 0; r < A; ++r) f[r] = gen(r);
        __builtin_amdgcn_sched_barrier(0);
        const float t1 = s_t[1];
        wmix<Z, 1>(f, t1, sg);
        wtrans<Z, 1, 0>(f, xb, o1, o0);
        wmix<Z, 0>(f, t1, sg);
        float sc = mu1;   // restores the norm: with the next phase
        if constexpr (PP == 3) {
            const float2* row = dyn + 4 * R + cd.base[2];
#pragma unroll
            for (int r = 0; r < A; ++r) {
                const float2 t = row[T[0].at(r)];
                f[r] = cmul(f[r], make_float2(sc * t.x, sc * t.y));
                if ((r & 7) == 7) __builtin_amdgcn_sched_barrier(0);
            }
            pmix(f, s_t[2], cd.mixed[2], sg);
            sc = static_cast<float>(sqrt(kpow(2)));
        }
#pragma unroll
        for (int r = 0; r < A; ++r) f[r] = make_float2(sc * f[r].x, sc * f[r].y);
        // ---- last layer on quadruples of qubits 0 and 1 (f' = D_p f, d0 = f'00 - f'11, s1 = f'01 + f'10):
        // <f'|M|f'> = ZZ - 2 cos sin Re(d0* s1) + sin^2 (|s1|^2 - |d0|^2); M f' = f'00 - w, f'11 + w,
        // v - f'01, v - f'10 with w = sin^2 d0 + cos sin s1, v = sin^2 s1 - cos sin d0.
        float2 lam[GRAD ? A : 1];
        double zv = 0.0, iv = 0.0, dv = 0.0;
        float gp = 0.f;
        {
            Tab<A>& TL = T[PP - 2];
            TL.opaque();
            const float2* row = dyn + (2 + PP) * R + cd.base[PP];
            const float cmid = static_cast<float>(cd.base[PP]) - cd.mid[PP];
#pragma unroll
            for (int q = 0; q < A; q += 4) {
                float2 t[4], d[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    t[i] = row[TL.at(q + i)];
                    d[i] = cmul(f[q + i], t[i]);
                    const double x = d[i].x, y = d[i].y;
                    if (i == 1 || i == 2) zv = fma(-y, y, fma(-x, x, zv));
                    else zv = fma(y, y, fma(x, x, zv));
                }
                const float2 d0 = make_float2(d[0].x - d[3].x, d[0].y - d[3].y);
                const float2 s1 = make_float2(d[1].x + d[2].x, d[1].y + d[2].y);
                const double ax = d0.x, ay = d0.y, bx = s1.x, by = s1.y;
                iv = fma(-ay, by, fma(-ax, bx, iv));
                dv = fma(by, by, fma(bx, bx, fma(-ay, ay, fma(-ax, ax, dv))));
                if constexpr (GRAD) {
                    const float2 w = make_float2(fmaf(ss2, d0.x, cs2 * s1.x), fmaf(ss2, d0.y, cs2 * s1.y));
                    const float2 v = make_float2(fmaf(ss2, s1.x, -cs2 * d0.x), fmaf(ss2, s1.y, -cs2 * d0.y));
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const float2 x = (i == 1 || i == 2) ? v : w;
                        const float2 m = i == 0 ? make_float2(d[i].x - x.x, d[i].y - x.y)
                                       : i == 3 ? make_float2(d[i].x + x.x, d[i].y + x.y)
                                                : make_float2(x.x - d[i].x, x.y - d[i].y);
                        // Im(conj(m) d) = -+ Im(conj(x) d): minus for 00, where m = d - x
                        const float im = i == 0 ? fmaf(x.y, d[i].x, -x.x * d[i].y) : fmaf(x.x, d[i].y, -x.y * d[i].x);
                        gp = fmaf(static_cast<float>(TL.at(q + i)) + cmid, im, gp);
                        lam[q + i] = cmulc(m, t[i]);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        Zs = fma(wt, zv, Zs);
        Is = fma(wt, iv, Is);
        Ds = fma(wt, dv, Ds);
        if constexpr (GRAD) {
            Wd = fma(e.dw, zv + 2.0 * s_cs[0] * s_cs[1] * iv + s_cs[1] * s_cs[1] * dv, Wd);
            Gp = fma(wt, static_cast<double>(gp), Gp);
            if constexpr (PP == 3) {
                const int m = cd.mixed[2];
                const double k2 = kpow(2);
                const float s = static_cast<float>(sqrt(k2));
                const float2 b2 = pxsum(f, lam, m, sg);
                B2 = fma(wt, static_cast<double>(b2.x) + static_cast<double>(b2.y), B2);
                pmix(f, -s_t[2], m, sg);
                pmix(lam, -s_t[2], m, sg);
                T[0].opaque();
                const float2* row = dyn + 4 * R + cd.base[2];
                const float cmid = static_cast<float>(cd.base[2]) - cd.mid[2];
                float ga = 0.f;
#pragma unroll
                for (int r = 0; r < A; ++r) {
                    const float2 t0 = row[T[0].at(r)];
                    const float2 t = make_float2(s * t0.x, s * t0.y);
                    const float im = fmaf(lam[r].x, f[r].y, -lam[r].y * f[r].x);
                    ga = fmaf(static_cast<float>(T[0].at(r)) + cmid, im, ga);
                    f[r] = cmulc(f[r], t);
                    lam[r] = cmulc(lam[r], t);
                    if ((r & 3) == 3) __builtin_amdgcn_sched_barrier(0);
                }
                G2 = fma(wt * k2, static_cast<double>(ga), G2);
            }
            // layer 1: the terms of qubits 0-7 behind it; then lambda alone is undone
            const float2 b1 = pxsum(f, lam, 8, sg);
            B1 = fma(wt, static_cast<double>(b1.x) + static_cast<double>(b1.y), B1);
            wmix<Z, 0>(lam, -t1, sg);
            wtrans<Z, 0, 1>(lam, xb, o0, o1);
            wmix<Z, 1>(lam, -t1, sg);
#pragma unroll
            for (int w = 0; w < A / 4; ++w) asm volatile("" : "+v"(k1[w]));
            float g1 = 0.f;
            const float cm = cd.mid[1];
#pragma unroll
            for (int r = 0; r < A; ++r) {
                f[r] = gen(r);
                const float im = fmaf(lam[r].x, f[r].y, -lam[r].y * f[r].x);
                g1 = fmaf(static_cast<float>(static_cast<int>(T1(r)) + ca[r & 3] + cb[r >> 2]) - cm, im, g1);
                if ((r & 3) == 3) __builtin_amdgcn_sched_barrier(0);
            }
            G1 = fma(wt, static_cast<double>(g1), G1);
            float bu = 0.f;
#pragma unroll
            for (int i = 0; i < Z::NR; ++i) bu += rdot_bit(i, f, lam);
            const float bur = bu;
            bu = 0.f;
            static_for<0, Z::NQ>([&](auto I) {
                constexpr int i = decltype(I)::value;
                float a0 = 0.f, a1 = 0.f;
#pragma unroll
                for (int r = 0; r < A; r += 4) row_dot4<i>(a0, a1, f, lam, r);
                bu = fmaf(sg[i], a0 + a1, bu);
            });
            B1u = fma(wt, static_cast<double>(bur) + static_cast<double>(bu), B1u);
        }
    }
    // psi is at its true norm times 2^(kin/2) behind layer 1; the undone layer scales lambda by 1 / mu_1
    const double n0 = cd.shell_norm * exp2(-static_cast<double>(KIN)), n1 = n0 * static_cast<double>(mu1);
    const double C = s_cs[0], S = s_cs[1];
    double v[8] = {n0 * (Zs + 2.0 * C * S * Is + S * S * Ds), 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    if constexpr (GRAD) {
        v[1] = n0 * 2.0 * (2.0 * (C * C - S * S) * Is + 2.0 * C * S * Ds);
        v[2] = 2.0 * n0 * Gp;
        v[3] = 2.0 * (n0 * B1 + n1 * B1u);
        v[4] = 2.0 * n1 * G1 + n0 * Wd;
        v[5] = 2.0 * n0 * B2;
        v[6] = 2.0 * n0 * G2;
        const double x = wave_sum8(v, lane);
        const int i = (lane & 8 ? 4 : 0) | (lane & 3);
        if ((lane & ~11) == 0) s_sum[tid >> 6][i] = x;
    } else {
        const double x = wave_sum(v[0]);
        if (lane == 0) s_sum[tid >> 6][0] = x;
    }
    __syncthreads();
    constexpr int NV = GRAD ? 2 * PP + 1 : 1;
    if (tid < NV) {
        double x = 0.0;
#pragma unroll
        for (int w = 0; w < NWV; ++w) x += s_sum[w][tid];
        // 0: <ZZ>; j >= 1: gradient entry j - 1 (gamma_1 .. p, beta_1 .. p)
        const int code = tid == 0 ? 0 : tid == 1 ? 2 * PP : tid == 2 ? PP : tid == 3 ? PP + 1 : tid == 4 ? 1
                       : tid == 5 ? PP + 2 : 2;
        a.part[(static_cast<size_t>(pt) * a.all_units + a.unit0 + un) * NV + code] = x;
    }
}

template <int KIN>
hipError_t launch_wide_k(bool grad, const WdArgs& a, hipStream_t st) {
    const int64_t blocks = static_cast<int64_t>(a.n_units) * a.P;
    if (blocks <= 0) return hipSuccess;
    // rows of the cone's own cut values: with those of the whole plan (up to 511 phases where cones have
    // couplings of opposite signs) 14 inner qubits would not fit the 160 KiB
    static_assert(Uz<KIN>::NPAD * sizeof(float2) + WD_CFG * sizeof(CfgWd) + Uz<KIN>::W + 512 +
                          ((3 + WD_PMAX) * WD_ROWS + 2 * WD_ROWS) * sizeof(float2) <= 160 * 1024,
                  "state, configurations, sums (a double per eight threads), phase rows, cosines");
    if (a.R > WD_ROWS || a.wz >= WD_ROWS) return hipErrorInvalidValue;
    const size_t lds = (static_cast<size_t>(3 + a.p) * a.R + 2 * (a.wz + 1)) * sizeof(float2);
    const dim3 grid(static_cast<unsigned>(blocks)), block(Uz<KIN>::W);
    if (a.p == 2) {
        if (grad) hipLaunchKernelGGL((k_wide<KIN, true, 2>), grid, block, lds, st, a);
        else hipLaunchKernelGGL((k_wide<KIN, false, 2>), grid, block, lds, st, a);
    } else {
        if (grad) hipLaunchKernelGGL((k_wide<KIN, true, 3>), grid, block, lds, st, a);
        else hipLaunchKernelGGL((k_wide<KIN, false, 3>), grid, block, lds, st, a);
    }
    return hipGetLastError();
}

}  // namespace qaoa
