// Light cones that hold the same qubits (small graphs, deep circuits: every cone is the whole
// graph) share one state: one simulation per (group, angle point) gives every member's <Z_u Z_v>,
// and one adjoint with the observable V = sum_m W_m [x_u != x_v] gives the gradient of their
// weighted sum (Sec. 3: E is linear in the terms).
//
// The state is stored on the K - 1 qubits below the last one (global flip, as in
// fused_impl.hpp), KL of them, A = 2^RB amplitudes per thread, in two layouts:
//   L0  registers: qubits 0 .. RB-1; 16-lane rows: the next ROW; the others above
//   L1  registers and, beyond them, row lanes exchanged with those others
// so one LDS transpose per layer brings every qubit into a register or a row, where it is mixed
// by butterflies or DPP operands, and the dropped qubit's mixer, which pairs y with its
// complement, rides on that transpose.  Amplitudes are held in the gauge i^|y|, in which the
// mixers of the stored qubits are real rotations (see inner_impl.hpp) and the dropped qubit's is
// phi_y += -i tau (-1)^|y| i^-KL phi_ybar.
//
// Layers alternate L0 -> L1 and L1 -> L0 so that the last one ends in L0.
#pragma once

#include "inner_impl.hpp"
#include "whole.hpp"

namespace qaoa {

template <int K_>
struct Wz {
    static constexpr int K = K_, KL = K - 1;
    static constexpr int RB = KL >= 12 ? 4 : 3;
    static constexpr int A = 1 << RB;
    static constexpr int TB = KL - RB;
    static constexpr int TPI = 1 << TB;                       // threads per item
    static constexpr int WG = TPI < 64 ? 64 : TPI;
    static constexpr int IPW = WG / TPI;
    static constexpr int ROW = TB < 4 ? TB : 4;
    static constexpr int REST = TB - ROW;                     // qubits above the rows in L0
    static constexpr int NR = REST < RB ? REST : RB;          // of them in registers in L1
    static constexpr int NQ = REST - NR;                      // and on row lanes
    static constexpr uint32_t N = 1u << KL;
    // qubit of register bit i, row lane i, upper thread bit i
    static constexpr int reg(int lay, int i) { return lay == 1 && i < NR ? RB + ROW + i : i; }
    static constexpr int row(int lay, int i) { return lay == 1 && i < NQ ? RB + ROW + NR + i : RB + i; }
    static constexpr int up(int lay, int i) { return lay == 0 ? RB + ROW + i : (i < NR ? i : RB + i - NR); }
    // padded LDS index of y, additive over its bits: the 16 lanes of a row hit 16 bank pairs in both
    // layouts (weights 1, 2, 4, 8 mod 16; the qubit that L1 puts on row lane 0 takes over the
    // weight of the one it displaces)
    static constexpr uint32_t wt(int j) {
        uint32_t w = (1u << j) + ((1u << j) >> 4);
        if (NQ > 0 && j == RB + ROW + NR) w += wt_row0();
        return w;
    }
    static constexpr uint32_t wt_row0() { return ((1u << RB) + ((1u << RB) >> 4)) & 15u; }
    static constexpr uint32_t PALL = [] {
        uint32_t s = 0;
        for (int j = 0; j < KL; ++j) s += wt(j);
        return s;
    }();
    static constexpr uint32_t NPAD = PALL + 1;
};

template <class Z, int LAY>
__host__ __device__ constexpr uint32_t wreg(int r) {          // basis index of register r
    uint32_t y = 0;
    for (int i = 0; i < Z::RB; ++i)
        if ((r >> i) & 1) y |= 1u << Z::reg(LAY, i);
    return y;
}
template <class Z, int LAY>
__host__ __device__ constexpr uint32_t wregp(int r) {         // its padded index
    uint32_t y = 0;
    for (int i = 0; i < Z::RB; ++i)
        if ((r >> i) & 1) y += Z::wt(Z::reg(LAY, i));
    return y;
}

// Thread coordinates: row qubits (logical) and upper bits.
struct WhThread {
    int xq[4];
    uint32_t up;
};
template <class Z>
__device__ __forceinline__ WhThread wh_thread(uint32_t tau) {
    WhThread t;
    const int b0 = tau & 1, b1 = (tau >> 1) & 1, b2 = (tau >> 2) & 1, b3 = (tau >> 3) & 1;
    t.xq[0] = Z::ROW > 2 ? b0 ^ b2 : b0;
    t.xq[1] = Z::ROW > 2 ? b1 ^ b2 : b1;
    t.xq[2] = Z::ROW > 3 ? b2 ^ b3 : b2;
    t.xq[3] = b3;
    t.up = tau >> Z::ROW;
    return t;
}
// the thread's basis index in a layout (padded: its LDS index)
template <class Z, int LAY, bool PAD>
__device__ __forceinline__ uint32_t wh_base(const WhThread& t) {
    uint32_t y = 0;
#pragma unroll
    for (int i = 0; i < Z::ROW; ++i) y += t.xq[i] ? (PAD ? Z::wt(Z::row(LAY, i)) : 1u << Z::row(LAY, i)) : 0u;
#pragma unroll
    for (int i = 0; i < Z::REST; ++i)
        y += ((t.up >> i) & 1u) ? (PAD ? Z::wt(Z::up(LAY, i)) : 1u << Z::up(LAY, i)) : 0u;
    return y;
}

// Real rotation of one pair (gauged mixer).
__device__ __forceinline__ void rot(float2& a, float2& b, float t) {
    const float2 a0 = a;
    a.x = fmaf(-t, b.x, a.x);
    a.y = fmaf(-t, b.y, a.y);
    b.x = fmaf(t, a0.x, b.x);
    b.y = fmaf(t, a0.y, b.y);
}

template <class Z, int LAY, int A>
__device__ __forceinline__ void wmix(float2 (&v)[A], float t, const float (&sg)[4]) {
#pragma unroll
    for (int i = 0; i < (LAY == 0 ? Z::RB : Z::NR); ++i) {
#pragma unroll
        for (int r = 0; r < A; ++r)
            if (!(r & (1 << i))) rot(v[r], v[r | (1 << i)], t);
        __builtin_amdgcn_sched_barrier(0);
    }
    static_for<0, (LAY == 0 ? Z::ROW : Z::NQ)>([&](auto I) {
        constexpr int i = decltype(I)::value;
        const float ts = t * sg[i];
#pragma unroll
        for (int r = 0; r < A; r += 4) row_rot4<i>(v[r], v[r + 1], v[r + 2], v[r + 3], ts);
    });
}

// Im <l| sum X_j |f> over the qubits that layout LAY mixes: FP32 over those in registers and over those of
// the row, FP64 beyond.
template <class Z, int LAY, int A>
__device__ __forceinline__ double wxsum(float2 (&f)[A], float2 (&l)[A], const float (&sg)[4]) {
    float acc = 0.f;
#pragma unroll
    for (int i = 0; i < (LAY == 0 ? Z::RB : Z::NR); ++i) {
        float a0 = 0.f, a1 = 0.f;
#pragma unroll
        for (int r = 0; r < A; ++r)
            if (!(r & (1 << i))) {
                const int s = r | (1 << i);
                a0 = fmaf(l[s].x, f[r].x, a0);
                a1 = fmaf(l[r].x, f[s].x, a1);
                a0 = fmaf(l[s].y, f[r].y, a0);
                a1 = fmaf(l[r].y, f[s].y, a1);
            }
        acc += a0 - a1;
        __builtin_amdgcn_sched_barrier(0);
    }
    const double sum = static_cast<double>(acc);
    acc = 0.f;
    static_for<0, (LAY == 0 ? Z::ROW : Z::NQ)>([&](auto I) {
        constexpr int i = decltype(I)::value;
        float a0 = 0.f, a1 = 0.f;
#pragma unroll
        for (int r = 0; r < A; r += 4) row_dot4<i>(a0, a1, f, l, r);
        acc = fmaf(sg[i], a0 + a1, acc);
    });
    return sum + static_cast<double>(acc);
}

// c b with c = i^-E.
template <int E>
__device__ __forceinline__ float2 ipow(float2 b) {
    if constexpr ((E & 3) == 0) return b;
    else if constexpr ((E & 3) == 1) return make_float2(b.y, -b.x);
    else if constexpr ((E & 3) == 2) return make_float2(-b.x, -b.y);
    else return make_float2(-b.y, b.x);
}

// Transpose FROM -> TO with the dropped qubit's mixer; sT: (-1)^|y| of the thread's part in TO.
template <class Z, int FROM, int TO, int A>
__device__ __forceinline__ void wpose(float2 (&v)[A], float2* xb, uint32_t of, uint32_t ot, float t, float sT) {
    __syncthreads();
#pragma unroll
    for (int r = 0; r < A; ++r) xb[of + wregp<Z, FROM>(r)] = v[r];
    __syncthreads();
    const float2* pt = xb + ot;
    const float2* pc = xb + (Z::PALL - wregp<Z, TO>(A - 1) - ot);
    const float ts = t * sT;
#pragma unroll
    for (int r = 0; r < A; ++r) {
        const float2 a = pt[wregp<Z, TO>(r)];
        const float2 b = ipow<Z::KL + 1>(pc[wregp<Z, TO>(A - 1 - r)]);
        const float s = (__builtin_popcount(r) & 1) ? -ts : ts;
        v[r] = make_float2(fmaf(s, b.x, a.x), fmaf(s, b.y, a.y));
    }
}

// The same undoing the mixer on psi and lambda; returns the thread's share of
// Im <l| X_(K-1) |f> on the values before the undo.
template <class Z, int FROM, int TO, int A>
__device__ __forceinline__ float wunpose2(float2 (&f)[A], float2 (&l)[A], float2* xa, float2* xc, uint32_t of,
                                          uint32_t ot, float t, float sT) {
    __syncthreads();
#pragma unroll
    for (int r = 0; r < A; ++r) {
        xa[of + wregp<Z, FROM>(r)] = f[r];
        xc[of + wregp<Z, FROM>(r)] = l[r];
    }
    __syncthreads();
    const uint32_t oc = Z::PALL - wregp<Z, TO>(A - 1) - ot;
    const float ts = -t * sT;
    float acc = 0.f;
#pragma unroll
    for (int r = 0; r < A; ++r) {
        const bool odd = (__builtin_popcount(r) & 1) != 0;
        const float s = odd ? -ts : ts;
        const float2 fa = xa[ot + wregp<Z, TO>(r)], la = xc[ot + wregp<Z, TO>(r)];
        const float2 fb = xa[oc + wregp<Z, TO>(A - 1 - r)], lb = xc[oc + wregp<Z, TO>(A - 1 - r)];
        const float2 x = ipow<Z::KL>(fb);   // without its sign: (X f)_y
        const float im = fmaf(la.x, x.y, -la.y * x.x);
        acc += odd ? -im : im;
        const float2 fr = ipow<Z::KL + 1>(fb), lr = ipow<Z::KL + 1>(lb);
        f[r] = make_float2(fmaf(s, fr.x, fa.x), fmaf(s, fr.y, fa.y));
        l[r] = make_float2(fmaf(s, lr.x, la.x), fmaf(s, lr.y, la.y));
        if ((r & 3) == 3) __builtin_amdgcn_sched_barrier(0);
    }
    return acc * sT;
}

// ODD: the depth is odd (the first layer then starts in L1).
template <int K, bool GRAD, bool ODD, bool RW>
__global__ void __launch_bounds__((Wz<K>::WG)) k_whole(WhArgs a) {
    using Z = Wz<K>;
    constexpr int A = Z::A, KL = Z::KL, NWV = Z::TPI / 64;
    __shared__ __attribute__((aligned(16))) float2 xbuf[(GRAD ? 2 : 1) * Z::IPW * Z::NPAD];
    // dynamic: per item tau_l (float), mu_l = |kappa_l|^K, phase rows [3 + p][rowcap] (layer 1 in four
    // gauges); then, items of more than one wave, partial sums [2p][waves]
    extern __shared__ float2 dyn[];
    const int tid = threadIdx.x;
    const int il = tid >> Z::TB;
    const uint32_t tau = static_cast<uint32_t>(tid) & (Z::TPI - 1);
    const int p = a.p, RC = RW ? 0 : a.rowcap;
    int64_t item = a.item0 + static_cast<int64_t>(blockIdx.x) * Z::IPW + il;
    const bool valid = item < a.n_items;
    if (!valid) item = a.n_items - 1;
    const int64_t slot = item / a.P;
    const int64_t point = item - slot * a.P;
    const GroupWh& gd = a.groups[slot];
    const size_t ip = (static_cast<size_t>(gd.inst) * a.gamma_P + point) * p;
    const size_t per = static_cast<size_t>(p) * 2 + static_cast<size_t>(3 + p) * RC;
    float2* mine = dyn + il * per;
    double* mk = reinterpret_cast<double*>(mine);             // [p] |kappa_l|^2
    float2* ml = mine + p;                                     // [p] (tau_l, mu_l)
    float2* rows = mine + 2 * p;
    double* dsum = reinterpret_cast<double*>(dyn + Z::IPW * per);
    const double delta = a.deltas[gd.inst];
    for (int l = static_cast<int>(tau); l < p; l += Z::TPI) {
        double s, c, t, k2;
        sincos(a.beta[ip + l], &s, &c);
        if (fabs(c) >= fabs(s)) {
            t = s / c;
            k2 = c * c;
        } else {
            t = -c / s;
            k2 = s * s;
        }
        mk[l] = k2;
        double m = 1.0;
        for (int e = 0; e < K; ++e) m *= k2;
        ml[l] = make_float2(static_cast<float>(t), static_cast<float>(sqrt(m)));
    }
    if constexpr (!RW) {
        const int n = gd.cut_range;
        for (int i = static_cast<int>(tau); i < p * n; i += Z::TPI) {
            const int l = i / n, j = i - l * n;
            double s, c;
            sincos(a.gamma[ip + l] * delta * static_cast<double>(a.cut_min + gd.cut_row + j), &s, &c);
            const float x = static_cast<float>(c), y = static_cast<float>(-s);
            if (l == 0) {
                rows[j] = make_float2(x, y);
                rows[RC + j] = make_float2(-y, x);
                rows[2 * RC + j] = make_float2(-x, -y);
                rows[3 * RC + j] = make_float2(y, -x);
            } else {
                rows[(3 + l) * RC + j] = make_float2(x, y);
            }
        }
    }
    const WhThread th = wh_thread<Z>(tau);
    float sg[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) sg[i] = th.xq[i] ? 1.f : -1.f;
    const uint32_t y0 = wh_base<Z, 0, false>(th), y1 = wh_base<Z, 1, false>(th);
    const uint32_t o0 = wh_base<Z, 0, true>(th), o1 = wh_base<Z, 1, true>(th);
    const int pc = __builtin_popcount(y0);                     // the same qubit values in both layouts' threads
    const float sT = (pc & 1) ? -1.f : 1.f;
    float2* xb = xbuf + il * Z::NPAD;
    float2* xb2 = xbuf + ((GRAD ? Z::IPW : 0) + il) * Z::NPAD;
    // cut values in both layouts: bytes packed four per register, or floats
    uint32_t pk[2][A / 4];
    float cf[RW ? 2 : 1][RW ? A : 1];
    if constexpr (RW) {
        const float* cut = reinterpret_cast<const float*>(a.cut) + gd.cut_off;
#pragma unroll
        for (int r = 0; r < A; ++r) {
            cf[0][r] = cut[y0 + wreg<Z, 0>(r)];
            cf[1][r] = cut[y1 + wreg<Z, 1>(r)];
        }
    } else {
        const uint8_t* cut = a.cut + gd.cut_off;
#pragma unroll
        for (int w = 0; w < A / 4; ++w) pk[0][w] = pk[1][w] = 0u;
#pragma unroll
        for (int r = 0; r < A; ++r) {
            pk[0][r >> 2] |= static_cast<uint32_t>(cut[y0 + wreg<Z, 0>(r)]) << (8 * (r & 3));
            pk[1][r >> 2] |= static_cast<uint32_t>(cut[y1 + wreg<Z, 1>(r)]) << (8 * (r & 3));
        }
    }
    const double* gam = a.gamma + ip;
    auto cutof = [&](auto LAY, int r) { return (pk[decltype(LAY)::value][r >> 2] >> (8 * (r & 3))) & 255u; };
    auto phase = [&](auto LAY, int l, int r) {                 // exp(-i gamma_(l+1) C)
        if constexpr (RW) return rphase(gam[l] * 0.31830988618379067154, cf[decltype(LAY)::value][r]);
        else return rows[(l ? 3 + l : 0) * RC + cutof(LAY, r)];
    };
    __syncthreads();

    float2 f[A];
    // D_1 |+>, gauged, without its norm 2^(-K/2)
    {
        using L = std::integral_constant<int, ODD ? 1 : 0>;
#pragma unroll
        for (int r = 0; r < A; ++r) {
            if constexpr (RW) {
                const float2 t = phase(L{}, 0, r);
                const int n = (pc + __builtin_popcount(r)) & 3;
                const float x = (n & 1) ? -t.y : t.x, y = (n & 1) ? t.x : t.y;
                f[r] = (n & 2) ? make_float2(-x, -y) : make_float2(x, y);
            } else {
                f[r] = rows[((pc + __builtin_popcount(r)) & 3) * RC + cutof(L{}, r)];
            }
        }
    }
    // layer l (0-based) from layout FROM to the other one
    auto layer = [&](auto FROM, int l) {
        constexpr int F = decltype(FROM)::value, T = 1 - F;
        const float t = ml[l].x;
        wmix<Z, F>(f, t, sg);
        wpose<Z, F, T>(f, xb, F ? o1 : o0, T ? o1 : o0, t, sT);
        wmix<Z, T>(f, t, sg);
        const float mu = ml[l].y;   // restores the norm: with the next phase, or alone after the last layer
        if (l + 1 < p) {
#pragma unroll
            for (int r = 0; r < A; ++r) {
                const float2 d = phase(std::integral_constant<int, T>{}, l + 1, r);
                f[r] = cmul(f[r], make_float2(mu * d.x, mu * d.y));
            }
        } else {
#pragma unroll
            for (int r = 0; r < A; ++r) f[r] = make_float2(mu * f[r].x, mu * f[r].y);
        }
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    int l = 0;
    if constexpr (ODD) layer(I1{}, l++);
    while (l < p) {
        layer(I0{}, l++);
        layer(I1{}, l++);
    }

    // ---- <Z_u Z_v> of every member: Walsh transform of the thread's probabilities over its
    // register qubits, then signed sums over the threads (|y|^2 over the half: doubled)
    const double hs = 2.0 * exp2(-static_cast<double>(K));
    {
        double w[A];
#pragma unroll
        for (int r = 0; r < A; ++r) {
            const double x = f[r].x, y = f[r].y;
            w[r] = fma(x, x, y * y);
        }
#pragma unroll
        for (int i = 0; i < Z::RB; ++i)
#pragma unroll
            for (int r = 0; r < A; ++r)
                if (!(r & (1 << i))) {
                    const double s = w[r] + w[r | (1 << i)], d = w[r] - w[r | (1 << i)];
                    w[r] = s;
                    w[r | (1 << i)] = d;
                }
        __syncthreads();
        double* wb = reinterpret_cast<double*>(xb);            // [A][TPI]
#pragma unroll
        for (int r = 0; r < A; ++r) wb[r * Z::TPI + tau] = w[r];
        __syncthreads();
        const MemWh* mem = a.mem + gd.mem_off;
        double* zz = a.zz + static_cast<size_t>(point) * a.M;
        auto sign = [&](uint32_t t, uint32_t m) {
            return (__builtin_popcount(wh_base<Z, 0, false>(wh_thread<Z>(t)) & m) & 1) != 0;
        };
        // qubit K - 1 of the stored half is 0
        auto mask = [&](const MemWh& x) { return ((1u << x.u) | (1u << x.v)) & (Z::N - 1u); };
        if constexpr (NWV >= 1) {
            for (int m = tid >> 6; m < gd.n_mem; m += NWV) {
                const uint32_t ms = mask(mem[m]);
                double s = 0.0;
                for (uint32_t t = tid & 63; t < static_cast<uint32_t>(Z::TPI); t += 64) {
                    const double x = wb[(ms & (A - 1)) * Z::TPI + t];
                    s += sign(t, ms) ? -x : x;
                }
                s = wave_sum(s);
                if ((tid & 63) == 0 && valid) zz[mem[m].orbit] = hs * s;
            }
        } else {
            for (int m = 0; m < gd.n_mem; ++m) {
                const uint32_t ms = mask(mem[m]);
                double s = wb[(ms & (A - 1)) * Z::TPI + tau];
                if (sign(tau, ms)) s = -s;
#pragma unroll
                for (int o = 1; o < Z::TPI; o <<= 1) s += __shfl_xor(s, o, 64);
                if (tau == 0 && valid) zz[mem[m].orbit] = hs * s;
            }
        }
    }
    if constexpr (GRAD) {
        double* g = a.g + static_cast<size_t>(point) * 2 * p * a.M;
        // entry j of dE/d(gamma, beta) through column rep: -2 dE (the sums weigh it by one)
        // (two entries at once: a wave's sum is six dependent steps of FP64 and lane moves)
        auto put = [&](int j0, double x0, int j1, double x1) {
            if constexpr (NWV >= 1) {
                const int lane = tid & 63, j = lane ? j1 : j0;
                const double x = wave_sum2(x0, x1, lane);
                if constexpr (NWV > 1) {
                    if (lane < 2) dsum[j * NWV + (tid >> 6)] = x;
                } else {
                    if (lane < 2 && valid) g[static_cast<size_t>(j) * a.M + gd.rep] = x;
                }
            } else {
#pragma unroll
                for (int o = 1; o < Z::TPI; o <<= 1) {
                    x0 += __shfl_xor(x0, o, 64);
                    x1 += __shfl_xor(x1, o, 64);
                }
                if (tau == 0 && valid) {
                    g[static_cast<size_t>(j0) * a.M + gd.rep] = x0;
                    g[static_cast<size_t>(j1) * a.M + gd.rep] = x1;
                }
            }
        };
        if (valid) {
            const MemWh* mem = a.mem + gd.mem_off;
            for (int i = static_cast<int>(tau); i < 2 * p * gd.n_mem; i += Z::TPI) {
                const int j = i / gd.n_mem, o = mem[i - j * gd.n_mem].orbit;
                if (o != gd.rep) g[static_cast<size_t>(j) * a.M + o] = 0.0;
            }
        }
        float2 lam[A];
        {
            const double* V = a.obs + gd.v_off + y0;
#pragma unroll
            for (int r = 0; r < A; ++r) {
                const double v = V[wreg<Z, 0>(r)];
                lam[r] = make_float2(static_cast<float>(v * f[r].x), static_cast<float>(v * f[r].y));
            }
        }
        const double sc = -2.0 * 2.0 * hs, unit = gd.scale;   // d<V> = 2 Im <lambda| . |psi>
        // undo layer l, which ended in layout END
        auto unlayer = [&](auto END, int l) {
            constexpr int F = decltype(END)::value, T = 1 - F;
            const float t = ml[l].x;
            const double k2 = mk[l];
            double b = wxsum<Z, F>(f, lam, sg);
            wmix<Z, F>(f, -t, sg);
            wmix<Z, F>(lam, -t, sg);
            double w = 1.0;   // every undone qubit scales the inner products by 1 / |kappa|^2
#pragma unroll
            for (int e = 0; e < (F == 0 ? Z::RB + Z::ROW : Z::NR + Z::NQ); ++e) w *= k2;
            b += w * static_cast<double>(wunpose2<Z, F, T>(f, lam, xb, xb2, F ? o1 : o0, T ? o1 : o0, t, sT));
            w *= k2;
            b += w * wxsum<Z, T>(f, lam, sg);
            wmix<Z, T>(f, -t, sg);
            wmix<Z, T>(lam, -t, sg);
            // gamma of the layer, from cut values less a constant (integers: their centre; real ones: the
            // table's): Im <lambda|psi> = Im <psi|V|psi> = 0 at every layer, V being real.  Both states
            // carry 1 / mu, which the undone phase takes back
            const float mu = ml[l].y;
            float ga = 0.f;
#pragma unroll
            for (int r = 0; r < A; ++r) {
                const float im = fmaf(lam[r].x, f[r].y, -lam[r].y * f[r].x);
                float c;
                if constexpr (RW) c = cf[T][r];
                else c = static_cast<float>(cutof(std::integral_constant<int, T>{}, r)) - gd.mid;
                ga = fmaf(c, im, ga);
                if (l > 0) {
                    const float2 d0 = phase(std::integral_constant<int, T>{}, l, r);
                    const float2 d = make_float2(mu * d0.x, mu * d0.y);
                    f[r] = cmulc(f[r], d);
                    lam[r] = cmulc(lam[r], d);
                }
            }
            put(p + l, sc * b * unit, l, sc * static_cast<double>(mu) * mu * static_cast<double>(ga) * unit);
        };
        int q = p - 1;
        while (q >= 1) {
            unlayer(I0{}, q--);
            unlayer(I1{}, q--);
        }
        if constexpr (ODD) unlayer(I0{}, 0);
        if constexpr (NWV > 1) {
            __syncthreads();
            for (int j = tid; j < 2 * p; j += Z::WG) {
                double x = 0.0;
                for (int w = 0; w < NWV; ++w) x += dsum[j * NWV + w];
                g[static_cast<size_t>(j) * a.M + gd.rep] = x;   // one item per workgroup: always valid
            }
        }
    }
}

template <int K>
size_t whole_dyn(int p, int rowcap, bool realw) {
    using Z = Wz<K>;
    const size_t per = static_cast<size_t>(p) * 2 + static_cast<size_t>(3 + p) * (realw ? 0 : rowcap);
    return Z::IPW * per * sizeof(float2) + (Z::TPI > 64 ? static_cast<size_t>(2 * p) * (Z::TPI / 64) * sizeof(double) : 0);
}

template <int K>
hipError_t launch_whole_k(bool grad, const WhArgs& a, hipStream_t st) {
    using Z = Wz<K>;
    const int64_t n = a.n_items - a.item0;
    if (n <= 0) return hipSuccess;
    const size_t dyn = whole_dyn<K>(a.p, a.rowcap, a.realw != 0);
    const bool odd = (a.p & 1) != 0;
    const int64_t blocks = (n + Z::IPW - 1) / Z::IPW;
    constexpr int64_t CH = static_cast<int64_t>(UINT32_MAX) / Z::WG;   // a grid holds fewer than 2^32 threads
    for (int64_t b0 = 0; b0 < blocks; b0 += CH) {
        const dim3 grid(static_cast<unsigned>(blocks - b0 < CH ? blocks - b0 : CH)), block(Z::WG);
        WhArgs c = a;
        c.item0 = a.item0 + b0 * Z::IPW;
#define QAOA_WH(G, O, R) hipLaunchKernelGGL((k_whole<K, G, O, R>), grid, block, dyn, st, c)
        if (a.realw) {
            if (grad) { if (odd) QAOA_WH(true, true, true); else QAOA_WH(true, false, true); }
            else { if (odd) QAOA_WH(false, true, true); else QAOA_WH(false, false, true); }
        } else {
            if (grad) { if (odd) QAOA_WH(true, true, false); else QAOA_WH(true, false, false); }
            else { if (odd) QAOA_WH(false, true, false); else QAOA_WH(false, false, false); }
        }
#undef QAOA_WH
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace qaoa
