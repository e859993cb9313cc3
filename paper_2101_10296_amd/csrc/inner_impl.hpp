// Light cones on their inner qubits, one wave per unit of work (p >= 2, up to 10 inner qubits).
//
// The reverse causal cone of Z_u Z_v (Sec. 2.3), taken layer by layer: behind layer l only
// operators on qubits closer than p - l + 1 to the edge are left, so the mixer of layer l
// cancels on every other qubit, and of its phase only couplings inside the qubits mixed by
// layer l - 1 remain (all couplings for l = 1).  The mixed qubits are a prefix, n_(p-l) of
// them, as the cone's qubits are sorted by distance.  The shell, the qubits at distance p, is
// never mixed: it stays in |+> and only shifts phases, so the term is the mean over its
// configurations y of a simulation of the kin = n_(p-1) inner qubits with layer-1 cut values
//   C_1(x; y) = C_in(x) + c(y) + sum_a x_a h_a(y).
// Leaves, shell qubits that couple to one inner qubit only, are two signs of that qubit whatever their
// number (shell.hpp).  Other shell qubits with equal couplings count by how many are 1 (t of m,
// weight binom(m, t)), and flipping every qubit of the cone pairs y with its complement: half of
// the configurations are run at twice the weight.  Where the cone has symmetries of its own (twins,
// u and v swapped), the configurations are listed up to them on the host (inner_plan.cpp).  A
// 26-qubit cone of a 4-regular graph at p = 2 (2 + 6 inner qubits, 18 leaves) is 10 states of 2^8
// amplitudes with 8 mixed qubits in place of 2^25 stored amplitudes with 26.  (At p = 2,
// trees have the closed form of depth2_impl.hpp.)
//
// Layout: A = 2^min(4, kin) amplitudes per lane (register bits: qubits 0..3), qubits 4..7 on
// the lanes of a 16-lane row, 8 and 9 on lane bits 4 and 5; a wave runs 64 >> (kin - 4)
// configurations at once.  Lane qubits are flipped by DPP moves that xor the lane with 1, 2,
// 7 and 15 (a basis of the row), and are held in the gauge i^x, where the mixer is a real
// rotation: re and im turn on their own, one FMA with a DPP operand per component, as cheap
// as a register butterfly.  Lane bits 4 and 5 are swapped with register bits (permlane
// swaps) for their butterflies.  No LDS transposes, no barriers inside the state.
//
// The last layer is taken in the Heisenberg picture: U^+ Z U = cos(2 beta) Z + sin(2 beta) Y
// on both qubits, so <ZZ>, its beta_p derivative and lambda = M f come from quadruples of
// amplitudes without a mixer, and the phase D_p is looked up once for its way there and back.
// The factored mixer (1 - i tau X) keeps |tau| <= 1; the X that the other branch of the
// factorisation leaves on the mixed prefix commutes with everything behind it (no couplings
// outside the prefix are left there).
//
// Bound: vector instruction issue (about 100 instructions per amplitude with the gradient at
// kin = 8, p = 2).  Measured on one MI355X against the statevector kernels that these cones ran
// on: energies of a random 4-regular n = 60, p = 2 (cones of up to 26 qubits, passes over device
// memory before) 5.27 -> 0.090 ms, with the leaves as signs 0.036; the 18-qubit cone of a torus at
// 32 points, with the gradient, 93 -> 23 us.
#pragma once

#include "fused_impl.hpp"
#include "inner.hpp"

namespace qaoa {

template <int KIN>
struct Iz {
    static constexpr int RB = KIN < 4 ? KIN : 4;        // register bits
    static constexpr int A = 1 << RB;
    static constexpr int LB = KIN - RB;                  // lane bits
    static constexpr int ROW = LB < 4 ? LB : 4;          // of them within a 16-lane row (gauged)
    static constexpr int CPW = 64 >> LB;                 // configurations per wave
};

struct alignas(16) CfgIn {   // one configuration of the shell
    int32_t h[8];
    int32_t c0;
    uint32_t z;
    double w;                // weight; 0 beyond the last configuration
};

template <int CTRL>
__device__ __forceinline__ float dppf(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xF, 0xF, true));
}
// lane xor 1, 2, 7, 15
template <int I>
__device__ __forceinline__ float row_flip(float x) {
    if constexpr (I == 0) return dppf<0xB1>(x);
    else if constexpr (I == 1) return dppf<0x4E>(x);
    else if constexpr (I == 2) return dppf<0x141>(x);
    else return dppf<0x140>(x);
}

// Sum over the wave (fixed order, the same in every lane).
__device__ __forceinline__ double wave_sum(double x) {
    auto step = [&](auto I) {
        constexpr int i = decltype(I)::value;
        const long long b = __double_as_longlong(x);
        const float lo = row_flip<i>(__int_as_float(static_cast<int>(b)));
        const float hi = row_flip<i>(__int_as_float(static_cast<int>(b >> 32)));
        const long long o = (static_cast<long long>(__float_as_int(hi)) << 32) |
                            static_cast<long long>(static_cast<unsigned>(__float_as_int(lo)));
        x += __longlong_as_double(o);
    };
    step(std::integral_constant<int, 0>{});
    step(std::integral_constant<int, 1>{});
    step(std::integral_constant<int, 2>{});
    step(std::integral_constant<int, 3>{});
    x += __shfl_xor(x, 16, 64);
    x += __shfl_xor(x, 32, 64);
    return x;
}

// Sums of eight values over the wave at once: value i lands in the lanes whose bits 0, 1 and 3 spell
// i.  Each of the first three steps halves the values a lane holds, where eight separate
// sums would take six steps each.
__device__ __forceinline__ double wave_sum8(double (&v)[8], int lane) {
    auto step = [&](auto I, int n, bool up) {   // keep the upper half of the values where up
        constexpr int i = decltype(I)::value;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (j >= n) continue;
            const double mine = up ? v[j + n] : v[j], other = up ? v[j] : v[j + n];
            const long long b = __double_as_longlong(other);
            float lo = __int_as_float(static_cast<int>(b)), hi = __int_as_float(static_cast<int>(b >> 32));
            if constexpr (i < 2) {
                lo = row_flip<i>(lo);
                hi = row_flip<i>(hi);
            } else {   // lane xor 8: rotate the row by 8
                lo = dppf<0x128>(lo);
                hi = dppf<0x128>(hi);
            }
            const long long o = (static_cast<long long>(__float_as_int(hi)) << 32) |
                                static_cast<long long>(static_cast<unsigned>(__float_as_int(lo)));
            v[j] = mine + __longlong_as_double(o);
        }
    };
    step(std::integral_constant<int, 2>{}, 4, (lane & 8) != 0);
    step(std::integral_constant<int, 1>{}, 2, (lane & 2) != 0);
    step(std::integral_constant<int, 0>{}, 1, (lane & 1) != 0);
    double x = v[0];
    x += __shfl_xor(x, 4, 64);
    x += __shfl_xor(x, 16, 64);
    x += __shfl_xor(x, 32, 64);
    return x;
}

// Two sums over the wave at once: a in the even lanes, b in the odd ones.
__device__ __forceinline__ double wave_sum2(double a, double b, int lane) {
    auto dpp = [](auto C, double x) {
        constexpr int c = decltype(C)::value;
        const long long v = __double_as_longlong(x);
        const float lo = dppf<c>(__int_as_float(static_cast<int>(v))), hi = dppf<c>(__int_as_float(static_cast<int>(v >> 32)));
        return __longlong_as_double((static_cast<long long>(__float_as_int(hi)) << 32) |
                                    static_cast<long long>(static_cast<unsigned>(__float_as_int(lo))));
    };
    const bool up = (lane & 1) != 0;
    double x = (up ? b : a) + dpp(std::integral_constant<int, 0xB1>{}, up ? a : b);   // lane xor 1
    x += dpp(std::integral_constant<int, 0x4E>{}, x);                                 // xor 2
    x += dpp(std::integral_constant<int, 0x124>{}, x);                                // row rotated by 4, 8
    x += dpp(std::integral_constant<int, 0x128>{}, x);
    x += __shfl_xor(x, 16, 64);
    x += __shfl_xor(x, 32, 64);
    return x;
}

// Exchange lane bit 4 (W32: 5) with register bit B (an involution).
template <bool W32, int B, int A>
__device__ __forceinline__ void lane_reg_swap(float2 (&v)[A]) {
#pragma unroll
    for (int r = 0; r < A; ++r)
        if (!(r & (1 << B))) {
            xswap(v[r].x, v[r | (1 << B)].x, W32);
            xswap(v[r].y, v[r | (1 << B)].y, W32);
        }
}

// a[i] += flip_I(a[i]) * t, and acc += flip_I(f[i]) * l[i], as FMAs with a DPP operand.  A DPP read
// of a register needs two wait states after its write; the block starts with them, and inside a
// block no instruction reads what another wrote (xdot's accumulators are no DPP operands).
#define QAOA_DPP0 "quad_perm:[1,0,3,2]"
#define QAOA_DPP1 "quad_perm:[2,3,0,1]"
#define QAOA_DPP2 "row_half_mirror"
#define QAOA_DPP3 "row_mirror"
#define QAOA_ROT4(D)                                                                     \
    asm volatile("s_nop 1\n"                                                             \
                 "v_fmac_f32_dpp %0, %0, %8 " D " row_mask:0xf bank_mask:0xf\n"          \
                 "v_fmac_f32_dpp %1, %1, %8 " D " row_mask:0xf bank_mask:0xf\n"          \
                 "v_fmac_f32_dpp %2, %2, %8 " D " row_mask:0xf bank_mask:0xf\n"          \
                 "v_fmac_f32_dpp %3, %3, %8 " D " row_mask:0xf bank_mask:0xf\n"          \
                 "v_fmac_f32_dpp %4, %4, %8 " D " row_mask:0xf bank_mask:0xf\n"          \
                 "v_fmac_f32_dpp %5, %5, %8 " D " row_mask:0xf bank_mask:0xf\n"          \
                 "v_fmac_f32_dpp %6, %6, %8 " D " row_mask:0xf bank_mask:0xf\n"          \
                 "v_fmac_f32_dpp %7, %7, %8 " D " row_mask:0xf bank_mask:0xf"            \
                 : "+v"(a.x), "+v"(a.y), "+v"(b.x), "+v"(b.y), "+v"(c.x), "+v"(c.y), "+v"(d.x), "+v"(d.y) \
                 : "v"(t))
template <int I>
__device__ __forceinline__ void row_rot4(float2& a, float2& b, float2& c, float2& d, float t) {
    if constexpr (I == 0) QAOA_ROT4(QAOA_DPP0);
    else if constexpr (I == 1) QAOA_ROT4(QAOA_DPP1);
    else if constexpr (I == 2) QAOA_ROT4(QAOA_DPP2);
    else QAOA_ROT4(QAOA_DPP3);
}
#define QAOA_DOT4(D)                                                                     \
    asm volatile("s_nop 1\n"                                                             \
                 "v_fmac_f32_dpp %0, %2, %10 " D " row_mask:0xf bank_mask:0xf\n"         \
                 "v_fmac_f32_dpp %1, %3, %11 " D " row_mask:0xf bank_mask:0xf\n"         \
                 "v_fmac_f32_dpp %0, %4, %12 " D " row_mask:0xf bank_mask:0xf\n"         \
                 "v_fmac_f32_dpp %1, %5, %13 " D " row_mask:0xf bank_mask:0xf\n"         \
                 "v_fmac_f32_dpp %0, %6, %14 " D " row_mask:0xf bank_mask:0xf\n"         \
                 "v_fmac_f32_dpp %1, %7, %15 " D " row_mask:0xf bank_mask:0xf\n"         \
                 "v_fmac_f32_dpp %0, %8, %16 " D " row_mask:0xf bank_mask:0xf\n"         \
                 "v_fmac_f32_dpp %1, %9, %17 " D " row_mask:0xf bank_mask:0xf"           \
                 : "+v"(a0), "+v"(a1)                                                    \
                 : "v"(f[r].x), "v"(f[r].y), "v"(f[r + 1].x), "v"(f[r + 1].y), "v"(f[r + 2].x), "v"(f[r + 2].y), \
                   "v"(f[r + 3].x), "v"(f[r + 3].y), "v"(l[r].x), "v"(l[r].y), "v"(l[r + 1].x), "v"(l[r + 1].y),  \
                   "v"(l[r + 2].x), "v"(l[r + 2].y), "v"(l[r + 3].x), "v"(l[r + 3].y))
template <int I, int A>
__device__ __forceinline__ void row_dot4(float& a0, float& a1, const float2 (&f)[A], const float2 (&l)[A], int r) {
    if constexpr (I == 0) QAOA_DOT4(QAOA_DPP0);
    else if constexpr (I == 1) QAOA_DOT4(QAOA_DPP1);
    else if constexpr (I == 2) QAOA_DOT4(QAOA_DPP2);
    else QAOA_DOT4(QAOA_DPP3);
}

// acc0 += Im(conj(la) pb) + Im(conj(lb) pa) of one pair of amplitudes, acc1 of another, in one block
// (single-instruction blocks cost a wait state each).
__device__ __forceinline__ void xacc2(float& a0, float& a1, float2 la, float2 lb, float2 pa, float2 pb, float2 lc,
                                      float2 ld, float2 pc, float2 pd) {
    asm volatile("v_fmac_f32 %0, %2, %9\n"
                 "v_fmac_f32 %1, %10, %17\n"
                 "v_fma_f32 %0, -%3, %8, %0\n"
                 "v_fma_f32 %1, -%11, %16, %1\n"
                 "v_fmac_f32 %0, %4, %7\n"
                 "v_fmac_f32 %1, %12, %15\n"
                 "v_fma_f32 %0, -%5, %6, %0\n"
                 "v_fma_f32 %1, -%13, %14, %1"
                 : "+v"(a0), "+v"(a1)
                 : "v"(la.x), "v"(la.y), "v"(lb.x), "v"(lb.y), "v"(pa.x), "v"(pa.y), "v"(pb.x), "v"(pb.y), "v"(lc.x),
                   "v"(lc.y), "v"(ld.x), "v"(ld.y), "v"(pc.x), "v"(pc.y), "v"(pd.x), "v"(pd.y));
}

// Mixer 1 - i t X on the first m qubits (FULL: all of them).  sg[i] = -1 / +1: the sign of the
// gauged rotation on row qubit i for a lane whose qubit is 0 / 1.
template <int KIN, bool FULL, int A>
__device__ __forceinline__ void in_mix(float2 (&v)[A], float t, int m, const float (&sg)[4]) {
    using Z = Iz<KIN>;
    auto reg_bit = [&](int i) {
        int nb = 0;
#pragma unroll
        for (int r = 0; r < A; ++r)
            if (!(r & (1 << i))) {
                bfly(v[r], v[r | (1 << i)], t);
                if ((++nb & 3) == 0) __builtin_amdgcn_sched_barrier(0);
            }
        __builtin_amdgcn_sched_barrier(0);
    };
#pragma unroll
    for (int i = 0; i < Z::RB; ++i)
        if (FULL || i < 2 || i < m) reg_bit(i);
    static_for<0, Z::ROW>([&](auto I) {
        constexpr int i = decltype(I)::value;
        if (FULL || 4 + i < m) {
            const float ts = t * sg[i];
#pragma unroll
            for (int r = 0; r < A; r += 4) row_rot4<i>(v[r], v[r + 1], v[r + 2], v[r + 3], ts);
        }
    });
    static_for<4, Z::LB>([&](auto I) {
        constexpr int i = decltype(I)::value;
        if (FULL || 4 + i < m) {
            lane_reg_swap<i == 5, 3>(v);
            reg_bit(3);
            lane_reg_swap<i == 5, 3>(v);
            __builtin_amdgcn_sched_barrier(0);
        }
    });
}

// Im <l| sum_(j < m) X_j |f>, this lane's share: FP32 over the register qubits and over those of the row
// (four each, as the stages of fused_impl.hpp), FP64 beyond.
template <int KIN, bool FULL, int A>
__device__ __forceinline__ double in_xsum(float2 (&f)[A], float2 (&l)[A], int m, const float (&sg)[4]) {
    using Z = Iz<KIN>;
    float acc = 0.f;
    auto reg_bit = [&](int i) {
        float a0 = 0.f, a1 = 0.f;
        const int o = i == 0 ? 2 : 1;   // the second pair of a block
#pragma unroll
        for (int r = 0; r < A; ++r)
            if (!(r & ((1 << i) | o))) {
                const int s = r | (1 << i), r2 = r | o, s2 = s | o;
                xacc2(a0, a1, l[r], l[s], f[r], f[s], l[r2], l[s2], f[r2], f[s2]);
            }
        acc += a0 + a1;
        __builtin_amdgcn_sched_barrier(0);
    };
#pragma unroll
    for (int i = 0; i < Z::RB; ++i)
        if (FULL || i < 2 || i < m) reg_bit(i);
    double sum = static_cast<double>(acc);
    acc = 0.f;
    static_for<0, Z::ROW>([&](auto I) {
        constexpr int i = decltype(I)::value;
        if (FULL || 4 + i < m) {
            float a0 = 0.f, a1 = 0.f;
#pragma unroll
            for (int r = 0; r < A; r += 4) row_dot4<i>(a0, a1, f, l, r);
            acc = fmaf(sg[i], a0 + a1, acc);
        }
    });
    if constexpr (Z::ROW > 0) sum += static_cast<double>(acc);
    acc = 0.f;
    static_for<4, Z::LB>([&](auto I) {
        constexpr int i = decltype(I)::value;
        if (FULL || 4 + i < m) {
            lane_reg_swap<i == 5, 3>(f);
            lane_reg_swap<i == 5, 3>(l);
            reg_bit(3);
            lane_reg_swap<i == 5, 3>(f);
            lane_reg_swap<i == 5, 3>(l);
            __builtin_amdgcn_sched_barrier(0);
        }
    });
    if constexpr (Z::LB > 4) sum += static_cast<double>(acc);
    return sum;
}

// The lane's table bytes of one layer (A of them, in register order).
template <int A>
struct Tab {
    uint32_t w[A / 4];
    __device__ __forceinline__ void load(const uint8_t* p) {
        if constexpr (A == 16) {
            const uint4 v = *reinterpret_cast<const uint4*>(p);
            w[0] = v.x; w[1] = v.y; w[2] = v.z; w[3] = v.w;
        } else {
            const uint2 v = *reinterpret_cast<const uint2*>(p);
            w[0] = v.x; w[1] = v.y;
        }
    }
    // keeps values derived from the table from being held in registers across its uses
    __device__ __forceinline__ void opaque() {
#pragma unroll
        for (int i = 0; i < A / 4; ++i) asm volatile("" : "+v"(w[i]));
    }
    __device__ __forceinline__ uint32_t at(int r) const { return (w[r >> 2] >> (8 * (r & 3))) & 255u; }
};

__device__ const double kBinom[30 * 30] = {
#include "binom30.inc"
};

// The configurations c .. of the next rounds, one per lane, for the lane groups that run them: mixed
// radix digits (how many of each group's qubits are 1), the first half of them at twice the weight,
// then the signs.
template <int KIN>
__device__ __forceinline__ void in_decode(CfgIn* cfg, const GrpIn* __restrict__ grp, int n_grp, uint32_t nc, uint32_t zmask,
                                          uint32_t c, int lane) {
    const uint32_t nh = (nc + 1) >> 1, n = nh << __builtin_popcount(zmask);
    uint32_t zz = c < n ? c / nh : 0u;
    uint32_t rem = c < n ? c - zz * nh : 0u;
    CfgIn e;
#pragma unroll
    for (int i = 0; i < 8; ++i) e.h[i] = 0;
    e.c0 = 0;
    e.z = 0;
    e.w = c < n ? (((nc & 1u) && rem == nh - 1) ? 1.0 : 2.0) : 0.0;
    for (uint32_t m = zmask; m; m &= m - 1, zz >>= 1) e.z |= (zz & 1u) << __builtin_ctz(m);
    for (int q = 0; q < n_grp; ++q) {
        const GrpIn& G = grp[q];
        const uint32_t d = static_cast<uint32_t>(G.m) + 1u;
        const uint32_t nx = rem / d;
        const int t = static_cast<int>(rem - nx * d);
        rem = nx;
        const int s = G.m - 2 * t;
        e.c0 += t * G.wsum;
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if (i + 2 < KIN) e.h[i] += s * G.h[i];
        e.w *= G.m < 4 ? ((t == 0 || t == G.m) ? 1.0 : static_cast<double>(G.m)) : kBinom[G.m * 30 + t];
    }
    __builtin_amdgcn_wave_barrier();
    cfg[lane] = e;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// The leaves' cosines, then the phase rows (layer 1 in four gauges, then layers 2..p), and the mixer
// factors of one point, by all threads of the workgroup.
__device__ __forceinline__ float2* in_phase(const InArgs& a, float2* dyn) { return dyn + (a.wz ? 2 * (a.wz + 1) : 0); }
inline size_t in_rows_bytes(const InArgs& a) {
    return (static_cast<size_t>(3 + a.p) * a.R + (a.wz ? 2 * (a.wz + 1) : 0)) * sizeof(float2);
}
struct InShared {
    float t[IN_PMAX + 1];
    double k2[IN_PMAX + 1];
    double cs[2];                 // cos, sin of 2 beta_p
};
__device__ __forceinline__ void in_rows(const InArgs& a, int p, int inst, int point, int tid, int threads, float2* dyn,
                                        InShared& sh) {
    const int R = a.R;
    double2* ct = reinterpret_cast<double2*>(dyn);
    dyn = in_phase(a, dyn);
    const size_t ip = (static_cast<size_t>(inst) * a.gamma_P + point) * p;
    const double delta = a.deltas[inst];
    for (int i = tid; i < p * R; i += threads) {
        const int l = i / R, j = i - l * R;
        double s, c;
        sincos(a.gamma[ip + l] * delta * static_cast<double>(a.cut_min + j), &s, &c);
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
    // on waves of their own, so that the three chains of FP64 sines run side by side
    const int o1 = threads > 64 ? 64 : 0, o2 = threads > 128 ? 128 : 0;
    if (a.wz && tid >= o1)
        for (int j = tid - o1; j <= a.wz; j += threads - o1)
            sincos(a.gamma[ip] * delta * static_cast<double>(j), &ct[j].y, &ct[j].x);
    if (const int i = tid - o2; i >= 0 && i < p) {   // exp(-i beta X) = kappa X^e (1 - i tau X), |tau| <= 1 (see k_tables)
        double s, c, t, k2;
        sincos(a.beta[ip + i], &s, &c);
        if (fabs(c) >= fabs(s)) {
            t = s / c;
            k2 = c * c;
        } else {
            t = -c / s;
            k2 = s * s;
        }
        sh.t[i + 1] = static_cast<float>(t);
        sh.k2[i + 1] = k2;
        if (i == p - 1) {
            sh.cs[0] = c * c - s * s;
            sh.cs[1] = 2.0 * s * c;
        }
    }
}

// What the units of a wave share: the lane's qubits.
template <int KIN>
struct InLane {
    int xq[6];
    float sg[4];
    uint32_t xl, gz;              // table offset of the lane; its gauge, qubits that are 1
    __device__ __forceinline__ explicit InLane(int lane) {
        using Z = Iz<KIN>;
        // row qubits of this lane: the lane is x0 1 ^ x1 2 ^ x2 7 ^ x3 15 in its 16-lane row
        const int b0 = lane & 1, b1 = (lane >> 1) & 1, b2 = (lane >> 2) & 1, b3 = (lane >> 3) & 1;
        xq[0] = Z::ROW > 2 ? b0 ^ b2 : b0;
        xq[1] = Z::ROW > 3 ? b1 ^ b2 : (Z::ROW > 2 ? b1 ^ b2 : b1);
        xq[2] = Z::ROW > 3 ? b2 ^ b3 : b2;
        xq[3] = b3;
        xq[4] = (lane >> 4) & 1;
        xq[5] = (lane >> 5) & 1;
        xl = 0;
        gz = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) sg[i] = xq[i] ? 1.f : -1.f;
#pragma unroll
        for (int i = 0; i < Z::LB; ++i) {
            xl |= static_cast<uint32_t>(xq[i]) << i;
            if (i < Z::ROW) gz += static_cast<uint32_t>(xq[i]);
        }
    }
};

// ---- last layer, quadruples of qubits 0 and 1 (f' = D_p f, s0 = f'00 + f'11, s1 = f'01 + f'10):
// <f'|M|f'> = ZZ + cos sin 2 Im(s0* s1) + sin^2 (|s1|^2 - |s0|^2) with cos, sin of 2 beta_p (sums
// zv, iv, dv); M f' = (f' - w, ...): w = sin^2 s0 + i cos sin s1 on 00, 11 and -(f' - w'),
// w' = sin^2 s1 + i cos sin s0 on 01, 10; l = D_p* M f', gp: the gamma_p derivative.
template <bool GRAD, int A, int AL>
__device__ __forceinline__ void in_last(const float2 (&f)[A], float2 (&l)[AL], const Tab<A>& T, const float2* row, float cmid,
                                        float cs2, float ss2, double& zv, double& iv, double& dv, float& gp) {
#pragma unroll
    for (int q = 0; q < A; q += 4) {
        float2 t[4], d[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            t[i] = row[T.at(q + i)];
            d[i] = cmul(f[q + i], t[i]);
            const double x = d[i].x, y = d[i].y;
            if (i == 1 || i == 2) zv = fma(-y, y, fma(-x, x, zv));
            else zv = fma(y, y, fma(x, x, zv));
        }
        const float2 s0 = make_float2(d[0].x + d[3].x, d[0].y + d[3].y);
        const float2 s1 = make_float2(d[1].x + d[2].x, d[1].y + d[2].y);
        const double ax = s0.x, ay = s0.y, bx = s1.x, by = s1.y;
        iv = fma(-ay, bx, fma(ax, by, iv));
        dv = fma(by, by, fma(bx, bx, fma(-ay, ay, fma(-ax, ax, dv))));
        if constexpr (GRAD) {
            const float2 w0 = make_float2(fmaf(ss2, s0.x, -cs2 * s1.y), fmaf(ss2, s0.y, cs2 * s1.x));
            const float2 w1 = make_float2(fmaf(ss2, s1.x, -cs2 * s0.y), fmaf(ss2, s1.y, cs2 * s0.x));
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const bool odd = i == 1 || i == 2;
                const float2 w = odd ? w1 : w0;
                const float2 m = odd ? make_float2(w.x - d[i].x, w.y - d[i].y)
                                     : make_float2(d[i].x - w.x, d[i].y - w.y);
                // Im(conj(m) d) = -+ Im(conj(w) d)
                const float im = odd ? fmaf(w.x, d[i].y, -w.y * d[i].x) : fmaf(w.y, d[i].x, -w.x * d[i].y);
                gp = fmaf(static_cast<float>(T.at(q + i)) + cmid, im, gp);
                l[q + i] = cmulc(m, t[i]);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

// Unit ch of a cone's `chunks` by one wave: put(0, <ZZ>), put(j, gradient entry j - 1).  PP = 2: depth
// 2, sums in registers; PP = 0: depth 3..IN_PMAX, sums per lane in lsum ([2p + 1][64]).  LISTED: the
// cone's configurations are listed (cfg is not used).  SIGNS: it has leaves.
template <int KIN, bool GRAD, int PP, bool LISTED, bool SIGNS, class Put>
__device__ __forceinline__ void in_unit(const InArgs& a, const ConeIn& cd, uint32_t ch, uint32_t chunks, int lane,
                                        const InLane<KIN>& ln, const float2* dyn0, const InShared& sh, CfgIn* cfg,
                                        double2* zfac, double* lsum, const Put& put) {
    using Z = Iz<KIN>;
    constexpr int A = Z::A;
    const int p = PP ? PP : a.p, R = a.R;
    const int (&xq)[6] = ln.xq;
    const float (&sg)[4] = ln.sg;
    const uint32_t xl = ln.xl, gz = ln.gz;
    const double2* ct = reinterpret_cast<const double2*>(dyn0);
    const float2* dyn = in_phase(a, const_cast<float2*>(dyn0));
    const float2* row1 = SIGNS ? dyn : dyn + (gz & 3u) * static_cast<uint32_t>(R);   // layer 1
    const float (&s_t)[IN_PMAX + 1] = sh.t;
    const double (&s_k2)[IN_PMAX + 1] = sh.k2;
    const double (&s_cs)[2] = sh.cs;
    const float cs2 = static_cast<float>(s_cs[0] * s_cs[1]), ss2 = static_cast<float>(s_cs[1] * s_cs[1]);
    const uint32_t nc = cd.nc;
    const bool listed = LISTED || cd.cfg_off >= 0;
    const uint32_t zmask = cd.zmask;
    const uint32_t nch = listed ? cd.n_cfg : ((nc + 1) >> 1) << __builtin_popcount(zmask);
    const uint32_t rounds = (nch + Z::CPW - 1) / Z::CPW;
    const uint32_t rp = (rounds + chunks - 1) / chunks;
    const uint32_t r0 = ch * rp, r1 = min(rounds, r0 + rp);
    const uint8_t* tab = a.tab + static_cast<size_t>(cd.tab_off) * 16 + (xl << Z::RB);
    constexpr uint32_t TS = (1u << KIN) < 16u ? 16u : (1u << KIN);   // bytes per table
    Tab<A> T;
    T.load(tab);
    // layer l's mixer prefix and scale |kappa_l|^m_l
    auto kpow = [&](int l) {
        double k = s_k2[l], x = 1.0;
        for (int e = PP == 2 ? KIN : cd.mixed[l]; e; e >>= 1) {
            if (e & 1) x *= k;
            k *= k;
        }
        return x;   // |kappa_l|^(2 m_l)
    };

    double Zs = 0.0, Is = 0.0, Ds = 0.0;              // <ZZ>, 2 Im, D of the last layer (see below)
    double Gp = 0.0, B1 = 0.0, G1 = 0.0;              // gamma_p, beta_(p-1) (PP = 2: beta_1), gamma_1
    double Wd = 0.0;                                  // gamma_1 through the weights
    if constexpr (SIGNS) {
        __builtin_amdgcn_wave_barrier();              // the last unit's weights are read
        z_factors(zmask, a.leaf, cd.z_off, ct, lane, zfac);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
    if constexpr (PP == 0 && GRAD)
        for (int i = 0; i < 2 * p + 1; ++i) lsum[i * 64 + lane] = 0.0;

    for (uint32_t r = r0; r < r1; ++r) {
        CfgIn e;
        if (listed) {
            const CfgList c = a.cfg[cd.cfg_off + r * Z::CPW + (lane >> Z::LB)];
#pragma unroll
            for (int i = 0; i < 8; ++i) e.h[i] = c.h[i];
            e.c0 = c.c0;
            e.z = c.z;
            e.w = c.w;
        } else {
            const uint32_t sub = (r - r0) % (64 / Z::CPW);
            if (sub == 0) in_decode<KIN>(cfg, a.grp + cd.grp_off, cd.n_grp, nc, zmask, r * Z::CPW + lane, lane);
            e = cfg[sub * Z::CPW + (lane >> Z::LB)];
        }
        double wt = e.w, dwt = 0.0;
        if constexpr (SIGNS) dwt = z_weight(zmask, e.z, zfac, wt);
        // row index of table value 0 in layer 1 for this lane, and the shifts of qubits 2, 3
        int lb = e.c0 + cd.base[1];
#pragma unroll
        for (int i = 0; i < Z::LB; ++i) lb += xq[i] ? e.h[i + 2] : 0;
        int cs[4], cb[4];   // without and with the gauge; the signs are two steps of it
        cs[0] = lb;
        cs[1] = lb + (KIN > 2 ? e.h[0] : 0);
        cs[2] = lb + (KIN > 3 ? e.h[1] : 0);
        cs[3] = cs[1] + cs[2] - lb;
        if constexpr (SIGNS) {
            const uint32_t g0 = gz + 2u * static_cast<uint32_t>(__builtin_popcount((e.z >> Z::RB) & xl));
            const uint32_t s2 = KIN > 2 ? (e.z >> 1) & 2u : 0u, s3 = KIN > 3 ? (e.z >> 2) & 2u : 0u;
#pragma unroll
            for (int i = 0; i < 4; ++i)
                cb[i] = cs[i] + static_cast<int>((g0 + (i & 1 ? s2 : 0u) + (i & 2 ? s3 : 0u)) & 3u) * R;
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) cb[i] = cs[i];
        }

        float2 f[A];
        {
#pragma unroll
            for (int q = 0; q < A; ++q) f[q] = row1[T.at(q) + cb[q >> 2]];
            __builtin_amdgcn_sched_barrier(0);
        }
        in_mix<KIN, true>(f, s_t[1], KIN, sg);
        float sc = 1.f;
        T.opaque();
        Tab<A> TL = T;
        if constexpr (PP == 0) {
            for (int l = 2; l < p; ++l) {
                const float s = static_cast<float>(sqrt(kpow(l - 1)));
                Tab<A> X;
                X.load(tab + (l - 2) * TS);
                const float2* row = dyn + (2 + l) * R + cd.base[l];
#pragma unroll
                for (int q = 0; q < A; ++q) {
                    const float2 t = row[X.at(q)];
                    f[q] = cmul(f[q], make_float2(s * t.x, s * t.y));
                    if ((q & 7) == 7) __builtin_amdgcn_sched_barrier(0);
                }
                in_mix<KIN, false>(f, s_t[l], cd.mixed[l], sg);
            }
            sc = static_cast<float>(sqrt(kpow(p - 1)));
#pragma unroll
            for (int q = 0; q < A; ++q) f[q] = make_float2(sc * f[q].x, sc * f[q].y);
            TL.load(tab + (p - 2) * TS);
        }
        float2 l[GRAD ? A : 1];
        double zv = 0.0, iv = 0.0, dv = 0.0;
        float gp = 0.f;
        in_last<GRAD>(f, l, TL, dyn + (2 + p) * R + cd.base[p], static_cast<float>(cd.base[p]) - cd.mid[p], cs2, ss2, zv, iv, dv,
                      gp);
        Zs = fma(wt, zv, Zs);
        Is = fma(wt, iv, Is);
        Ds = fma(wt, dv, Ds);
        if constexpr (GRAD) {
            if constexpr (SIGNS) Wd = fma(dwt, zv + 2.0 * s_cs[0] * s_cs[1] * iv + s_cs[1] * s_cs[1] * dv, Wd);
            Gp = fma(wt, static_cast<double>(gp), Gp);
            if constexpr (PP == 0) {
                for (int ly = p - 1; ly >= 2; --ly) {
                    const int m = cd.mixed[ly];
                    const double k2 = kpow(ly);
                    const float s = static_cast<float>(sqrt(k2));
                    const double b = in_xsum<KIN, false>(f, l, m, sg);
                    lsum[(p + ly) * 64 + lane] = fma(wt, b, lsum[(p + ly) * 64 + lane]);
                    in_mix<KIN, false>(f, -s_t[ly], m, sg);
                    in_mix<KIN, false>(l, -s_t[ly], m, sg);
                    Tab<A> X;
                    X.load(tab + (ly - 2) * TS);
                    const float2* row = dyn + (2 + ly) * R + cd.base[ly];
                    const float cmid = static_cast<float>(cd.base[ly]) - cd.mid[ly];
                    float ga = 0.f;
#pragma unroll
                    for (int q = 0; q < A; ++q) {
                        const float2 t0 = row[X.at(q)];
                        const float2 t = make_float2(s * t0.x, s * t0.y);
                        const float im = fmaf(l[q].x, f[q].y, -l[q].y * f[q].x);
                        ga = fmaf(static_cast<float>(X.at(q)) + cmid, im, ga);
                        f[q] = cmulc(f[q], t);
                        l[q] = cmulc(l[q], t);
                        if ((q & 3) == 3) __builtin_amdgcn_sched_barrier(0);
                    }
                    lsum[ly * 64 + lane] = fma(wt * k2, static_cast<double>(ga), lsum[ly * 64 + lane]);
                }
            }
            B1 = fma(wt, in_xsum<KIN, true>(f, l, KIN, sg), B1);
            in_mix<KIN, true>(l, -s_t[1], KIN, sg);
            float g1 = 0.f;
            T.opaque();
            {
                float cf[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) cf[i] = static_cast<float>(cs[i]) - cd.mid[1];
#pragma unroll
                for (int q = 0; q < A; ++q) {
                    const float2 t = row1[T.at(q) + cb[q >> 2]];
                    const float im = fmaf(l[q].x, t.y, -l[q].y * t.x);
                    g1 = fmaf(static_cast<float>(T.at(q)) + cf[q >> 2], im, g1);
                    if ((q & 7) == 7) __builtin_amdgcn_sched_barrier(0);
                }
            }
            G1 = fma(wt, static_cast<double>(g1), G1);
        }
    }
    // ---- the unit's sums: |psi|^2 carries 2^kin (generation without its norm) and, with PP = 2,
    // 1 / |kappa_1|^(2 kin); the undone layer 1 scales lambda by 1 / |kappa_1|^kin (PP = 0)
    const double n0 = cd.shell_norm * exp2(-static_cast<double>(KIN));
    const double k1 = kpow(1);
    const double nz = PP == 2 ? n0 * k1 : n0;
    const double n1 = PP == 2 ? nz : n0 * sqrt(k1);
    const double C = s_cs[0], S = s_cs[1];
    // linear in the last layer's three sums, so combined per lane before the wave's sum
    double v[8] = {nz * (Zs + 2.0 * C * S * Is + S * S * Ds), 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    if constexpr (GRAD) {
        v[1] = nz * 2.0 * (2.0 * (C * C - S * S) * Is + 2.0 * C * S * Ds);
        v[2] = 2.0 * nz * Gp;
        v[3] = 2.0 * nz * B1;
        v[4] = 2.0 * n1 * G1 + nz * Wd;
        const double x = wave_sum8(v, lane);
        const int i = (lane & 8 ? 4 : 0) | (lane & 2) | (lane & 1);   // the value that this lane holds
        if ((lane & ~11) == 0 && i < 5) put(i == 0 ? 0 : i == 1 ? 2 * p : i == 2 ? p : i == 3 ? p + 1 : 1, x);
        if constexpr (PP == 0) {
            for (int ly = 2; ly < p; ++ly) {
                const double ga = wave_sum(lsum[ly * 64 + lane]), be = wave_sum(lsum[(p + ly) * 64 + lane]);
                if (lane == 0) {
                    put(ly, 2.0 * n0 * ga);
                    put(p + ly, 2.0 * n0 * be);
                }
            }
        }
    } else {
        const double x = wave_sum(v[0]);
        if (lane == 0) put(0, x);
    }
}

// The segment of one instance that holds workgroup blk of `per` units, and its units u0 .. u1 - 1.
__device__ __forceinline__ void in_segment(const InArgs& a, int blk, int per, int& u0, int& u1, int& inst) {
    u0 = blk * per;
    u1 = a.units;
    inst = a.inst0;
    if (a.n_seg > 1) {
        const int32_t* sb = a.seg + a.n_seg + 1;
        int lo = 0, hi = a.n_seg;
        while (hi - lo > 1) {
            const int mid = (lo + hi) / 2;
            if (sb[mid] <= blk) lo = mid; else hi = mid;
        }
        u0 = a.seg[lo] + (blk - sb[lo]) * per;
        u1 = a.seg[lo + 1];
        inst = a.seg[2 * (a.n_seg + 1) + lo];
    }
}

template <int KIN, bool GRAD, int PP, bool SIGNS>
__global__ void __launch_bounds__(256, GRAD && PP == 0 ? 2 : 4) k_inner(InArgs a) {
    extern __shared__ __attribute__((aligned(16))) float2 dyn[];   // cosines and phase rows (in_rows); then (PP = 0) sums
    __shared__ CfgIn cfg_all[4][64];
    __shared__ InShared sh;
    __shared__ double2 s_z[4][16];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int p = PP ? PP : a.p, R = a.R;
    const int point = blockIdx.x / a.blocks + a.point0;
    const int blk = blockIdx.x % a.blocks;
    int u0, u1, inst;
    in_segment(a, blk, 4 * a.upw, u0, u1, inst);
    in_rows(a, p, inst, point, tid, 256, dyn, sh);
    __syncthreads();

    const InLane<KIN> ln(lane);
    double* lsum = nullptr;   // PP = 0: [2p + 1][64] sums of this wave's lanes
    if constexpr (PP == 0) lsum = reinterpret_cast<double*>(in_phase(a, dyn) + (3 + p) * R + ((3 + p) * R & 1)) + wave * (2 * p + 1) * 64;
    const int first = u0 + wave * a.upw;
    const int last = min(first + a.upw, u1);
    const int nv = GRAD ? 2 * p + 1 : 1;
    for (int uu = first; uu < last; ++uu) {
        const int u = __builtin_amdgcn_readfirstlane(uu);
        const int slot = u / a.chunks, ch = u - slot * a.chunks;
        const ConeIn& cd = a.cones[slot];
        double* out = a.chunks > 1 ? a.part + (static_cast<size_t>(point - a.point0) * a.units + u) * nv : nullptr;
        in_unit<KIN, GRAD, PP, false, SIGNS>(a, cd, ch, a.chunks, lane, ln, dyn, sh, cfg_all[wave], s_z[wave], lsum, [&](int code, double x) {
            if (out) out[code] = x;
            else if (code == 0) a.zz[static_cast<size_t>(point) * a.M + cd.orbit] = x;
            else a.g[(static_cast<size_t>(point) * 2 * p + (code - 1)) * a.M + cd.orbit] = x;
        });
    }
}

template <int KIN>
hipError_t launch_inner_k(bool grad, const InArgs& a, hipStream_t st) {
    const int64_t blocks = static_cast<int64_t>(a.blocks) * a.P;
    if (blocks <= 0) return hipSuccess;
    size_t lds = in_rows_bytes(a);
    if (a.p > 2 && grad) lds += 8 + 4 * static_cast<size_t>(2 * a.p + 1) * 64 * sizeof(double);
    const dim3 grid(static_cast<unsigned>(blocks)), block(256);
    auto go = [&](auto S) {
        constexpr bool SIGNS = decltype(S)::value;
        if (a.p == 2) {
            if (grad) hipLaunchKernelGGL((k_inner<KIN, true, 2, SIGNS>), grid, block, lds, st, a);
            else hipLaunchKernelGGL((k_inner<KIN, false, 2, SIGNS>), grid, block, lds, st, a);
        } else if constexpr (KIN >= 4) {   // p >= 3 leaves at least four inner qubits
            if (grad) hipLaunchKernelGGL((k_inner<KIN, true, 0, SIGNS>), grid, block, lds, st, a);
            else hipLaunchKernelGGL((k_inner<KIN, false, 0, SIGNS>), grid, block, lds, st, a);
        } else {
            return hipErrorInvalidValue;
        }
        return hipGetLastError();
    };
    return a.signs ? go(std::true_type{}) : go(std::false_type{});
}

}  // namespace qaoa
