// Small kernels around the light-cone kernels: per-call angle tables, per-plan cut
// tables, and the orbit-weighted combination of term values into E and dE.
#include <algorithm>

#include "device.hpp"
#include "inner.hpp"

namespace qaoa {

// phase[(i*p + l)*R + j] = exp(-i gamma_{i,l} delta c), c = cmin + j  (U_P on a basis state
// whose cut is delta c, cut values counted in the weight unit delta of the point's instance;
// Sec. 2.2 / 2.4, weights as in Sec. 4), computed in FP64 and rounded to FP32; rows i*p + l
// run over the instances' points (pl_per_inst rows per instance);
// mix[i*p + l] = (tau, |kappa|^2) of exp(-i beta_{i,l} X) = kappa X^e (1 - i tau X) (Sec. 2.2):
// tau = tan beta, |kappa|^2 = cos^2 beta when |cos beta| >= |sin beta|, otherwise
// tau = -cot beta, |kappa|^2 = sin^2 beta.
__global__ void k_tables(const double* __restrict__ gamma, const double* __restrict__ beta,
                         int64_t n_pl, int32_t R, int32_t cmin, const double* __restrict__ deltas,
                         int64_t pl_per_inst, float2* __restrict__ phase, float2* __restrict__ mix) {
    const int64_t total = n_pl * R;
    for (int64_t t = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; t < total;
         t += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        const int64_t pl = t / R;
        const int32_t j = static_cast<int32_t>(t - pl * R);
        const double delta = deltas[pl / pl_per_inst];
        double s, c;
        sincos(gamma[pl] * delta * static_cast<double>(cmin + j), &s, &c);
        phase[t] = make_float2(static_cast<float>(c), static_cast<float>(-s));
        if (j == 0) {
            // exp(-i beta X) = kappa X^e (1 - i tau X): the bounded factorisation
            double sb, cb;
            sincos(beta[pl], &sb, &cb);
            double t, k2;
            if (fabs(cb) >= fabs(sb)) {
                t = sb / cb;
                k2 = cb * cb;
            } else {
                t = -cb / sb;
                k2 = sb * sb;
            }
            mix[pl] = make_float2(static_cast<float>(t), static_cast<float>(k2));
        }
    }
}

// Tables of a new plan (integer weights), which its first call waits for.  One launch for both kinds, as cones
// in two forms have both.  A first call at p = 2 on a 20-node graph, 81 us with the inner tables alone: 22
// more for cut tables on a workgroup of 256 threads a cone with each edge read from memory, 6 more in
// parts with edges in LDS, 1 more in the same launch.
constexpr int CUT_EDGES = 14 * 13 / 2;   // different pairs of a workgroup-resident cone's qubits

// Cut table of a cone: table[x] = C(x) - cut_min for every basis state x of its k qubits,
// C(x) = sum over cone edges (a, b) of w_ab [x_a != x_b]  (MaxCut cost, Sec. 2.4).  Bound by latency where
// cones are few: a lane's four entries read each edge once, from LDS (k >= 2: entries come in fours),
// and few cones are spread in parts of 256 entries.
__device__ __forceinline__ void cut_table(const ConeDev& cd, uint32_t part, uint32_t parts, const PlanTabs& a) {
    __shared__ int32_t edge[CUT_EDGES];   // ends and weight, which a table of bytes bounds by 255
    const uint32_t N = 1u << cd.k;
    if (part * 256u >= N) return;
    const int32_t n = cd.n_edges < CUT_EDGES ? cd.n_edges : CUT_EDGES;
    for (int32_t e = threadIdx.x; e < n; e += 64)
        edge[e] = a.ea[cd.edge_off + e] | a.eb[cd.edge_off + e] << 8 | a.ew[cd.edge_off + e] * 65536;
    __syncthreads();
    uint8_t* out = a.cut + cd.cut_off;
    for (uint32_t x = part * 256u + threadIdx.x * 4u; x < N; x += parts * 256u) {
        int32_t c[4] = {-cd.cut_min, -cd.cut_min, -cd.cut_min, -cd.cut_min};
#pragma unroll 4
        for (int32_t e = 0; e < n; ++e) {
            const int32_t q = edge[e], i = q & 255, j = (q >> 8) & 255, w = q >> 16;
#pragma unroll
            for (uint32_t y = 0; y < 4; ++y) c[y] += w * static_cast<int32_t>((((x + y) >> i) ^ ((x + y) >> j)) & 1u);
        }
        uint32_t v = 0;
#pragma unroll
        for (int y = 0; y < 4; ++y) v |= static_cast<uint32_t>(static_cast<uint8_t>(c[y])) << (8 * y);
        *reinterpret_cast<uint32_t*>(out + x) = v;   // cut_off: a multiple of 16
    }
}

// Table of layer l of a cone on its inner qubits: the cut of the couplings inside the qubits mixed by layer
// l - 1, minus its smallest value.  In parts where the cones alone leave the chip idle (one workgroup
// took 60 us for the four tables of a ring's 10 inner qubits).
__device__ __forceinline__ void inner_table(const ConeIn& cd, int l, uint32_t part, uint32_t parts, const PlanTabs& a) {
    const uint32_t n = 1u << cd.kin, ts = n < 16u ? 16u : n;
    uint8_t* out = a.tab + static_cast<size_t>(cd.tab_off) * 16 + static_cast<size_t>(l - 2) * ts;
    const int m = cd.mixed[l - 1], cmin = cd.base[l] + a.cut_min;
    for (uint32_t x = part * 64u + threadIdx.x; x < ts; x += parts * 64u) {
        int32_t c = 0;
        for (int32_t e = 0; e < cd.n_edges; ++e) {
            const int32_t i = a.ea[cd.edge_off + e], j = a.eb[cd.edge_off + e];
            if (j < m) c += a.ew[cd.edge_off + e] * static_cast<int32_t>(((x >> i) ^ (x >> j)) & 1u);
        }
        out[x] = static_cast<uint8_t>(x < n ? c - cmin : 0);
    }
}

// cut_parts workgroups for each of n_cones cones, then in_parts for each layer 2 .. p of n_in inner ones
__global__ void __launch_bounds__(64) k_plan_tables(PlanTabs a) {
    uint32_t b = blockIdx.x;
    const uint32_t cuts = static_cast<uint32_t>(a.n_cones) * a.cut_parts;
    if (b < cuts) {
        cut_table(a.cones[b / a.cut_parts], b % a.cut_parts, a.cut_parts, a);
        return;
    }
    b -= cuts;
    const uint32_t t = b / a.in_parts, layers = static_cast<uint32_t>(a.p - 1);
    inner_table(a.in[t / layers], 2 + static_cast<int>(t % layers), b % a.in_parts, a.in_parts, a);
}

// Real-weight cut table of cone c over the stored half (qubit k-1 = 0 for k >= 3):
// table[x] = C(x) - c0 as a float, C(x) = sum over cone edges of w_ab [x_a != x_b] summed
// in FP64 (MaxCut cost with real couplings, Sec. 2.4 and Sec. 4).
__global__ void k_cut_tables_real(const ConeDev* __restrict__ cones, const int32_t* __restrict__ ea,
                                  const int32_t* __restrict__ eb, const double* __restrict__ ew,
                                  float* __restrict__ tables) {
    const ConeDev cd = cones[blockIdx.x];
    const uint32_t N = 1u << (cd.k >= 3 ? cd.k - 1 : cd.k);
    float* out = tables + cd.cut_off;
    for (uint32_t x = threadIdx.x; x < N; x += blockDim.x) {
        double c = 0.0;
        for (int32_t e = 0; e < cd.n_edges; ++e) {
            const int32_t a = ea[cd.edge_off + e], b = eb[cd.edge_off + e];
            if (((x >> a) ^ (x >> b)) & 1u) c += ew[cd.edge_off + e];
        }
        out[x] = static_cast<float>(c - static_cast<double>(cd.c0));
    }
}

hipError_t launch_cut_tables_real(const ConeDev* cones, int64_t n_cones, const int32_t* ea, const int32_t* eb,
                                  const double* ew, float* tables, hipStream_t st) {
    constexpr int64_t CH = static_cast<int64_t>(UINT32_MAX) / 256;
    for (int64_t c0 = 0; c0 < n_cones; c0 += CH) {
        const unsigned nx = static_cast<unsigned>(n_cones - c0 < CH ? n_cones - c0 : CH);
        hipLaunchKernelGGL(k_cut_tables_real, dim3(nx), dim3(256), 0, st, cones + c0, ea, eb, ew, tables);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// Per (instance j, point i) block, over the orbits m of instance j:
// block y == 0: energy = sum_m W_m (1 - zz[i][m]) / 2            (Sec. 3 reduced sum)
// block y == 1 + l: -1/2 sum_m Wg_m g[i][l][m] -> dgamma (l < p, times the instance's weight
// unit: cut values are counted in it) or dbeta (l >= p).
// Term rows i run over the Pc points of this call's chunk; results go to point i0 + i of an
// output with P_out points per instance.  Blocks b0 + blockIdx.x = j * Pc + i.
// Fixed-order reduction (deterministic): thread t sums m = t, t + 256, ...; then a tree.
// Bound by the latency of the loads where blocks are few: seven graphs of 9000 to 563 orbits at 8
// points 12.8 us one pair of loads after the other, 6.4 with eight pairs in flight.
__global__ void __launch_bounds__(256)
k_combine(const double* __restrict__ W, const double* __restrict__ Wg, const double* __restrict__ zz, const double* __restrict__ g,
          int32_t M, int32_t p, const int64_t* __restrict__ inst_orbit, const double* __restrict__ deltas,
          int64_t Pc, int64_t P_out, int64_t i0, int64_t b0, double* __restrict__ energy,
          double* __restrict__ dgamma, double* __restrict__ dbeta) {
    __shared__ double sh[256];
    const int64_t b = b0 + blockIdx.x;
    const int64_t j = b / Pc;
    const int64_t i = b - j * Pc;
    const int y = blockIdx.y;
    const double* src = (y == 0) ? zz + static_cast<size_t>(i) * M
                                 : g + (static_cast<size_t>(i) * 2 * p + (y - 1)) * M;
    const int64_t m0 = inst_orbit[j], m1 = inst_orbit[j + 1];
    double acc = 0.0;
    const double* w = y == 0 ? W : Wg;
    int64_t m = m0 + threadIdx.x;
    auto add = [&](double wm, double x) { acc += (y == 0) ? wm * (1.0 - x) * 0.5 : -0.5 * wm * x; };
    for (; m + 7 * 256 < m1; m += 8 * 256) {   // sixteen loads in flight, added in order
        double a[8], b[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            a[q] = w[m + q * 256];
            b[q] = src[m + q * 256];
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) add(a[q], b[q]);
    }
    for (; m < m1; m += 256) add(w[m], src[m]);
    sh[threadIdx.x] = acc;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (threadIdx.x < s) sh[threadIdx.x] += sh[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const size_t o = static_cast<size_t>(j) * P_out + i0 + i;
        if (y == 0) energy[o] = sh[0];
        else if (y - 1 < p) dgamma[o * p + (y - 1)] = deltas[j] * sh[0];
        else dbeta[o * p + (y - 1 - p)] = sh[0];
    }
}

// The same for instances of at most 64 orbits: a wave per (instance, point, value), the tree by lane
// moves (the larger workgroup's threads beyond the orbits hold zeros: same bits).  18 orbits, 17 values,
// 256 points: 5.4 us in workgroups of 256 threads each, 4.6 here.
__global__ void __launch_bounds__(256)
k_combine_small(const double* __restrict__ W, const double* __restrict__ Wg, const double* __restrict__ zz,
                const double* __restrict__ g, int32_t M, int32_t p, const int64_t* __restrict__ inst_orbit,
                const double* __restrict__ deltas, int64_t Pc, int64_t P_out, int64_t i0, int64_t t0, int64_t n, int32_t ny,
                double* __restrict__ energy, double* __restrict__ dgamma, double* __restrict__ dbeta) {
    const int64_t t = t0 + blockIdx.x * int64_t{4} + (threadIdx.x >> 6);
    if (t >= n) return;
    const int lane = threadIdx.x & 63;
    const int64_t b = t / ny;
    const int y = static_cast<int>(t - b * ny);
    const int64_t j = b / Pc, i = b - j * Pc;
    const double* src = (y == 0) ? zz + static_cast<size_t>(i) * M : g + (static_cast<size_t>(i) * 2 * p + (y - 1)) * M;
    const int64_t m = inst_orbit[j] + lane;
    double x = 0.0;
    if (m < inst_orbit[j + 1]) x = (y == 0) ? W[m] * (1.0 - src[m]) * 0.5 : -0.5 * Wg[m] * src[m];
#pragma unroll
    for (int s = 32; s > 0; s >>= 1) x += __shfl_down(x, s, 64);
    if (lane == 0) {
        const size_t o = static_cast<size_t>(j) * P_out + i0 + i;
        if (y == 0) energy[o] = x;
        else if (y - 1 < p) dgamma[o * p + (y - 1)] = deltas[j] * x;
        else dbeta[o * p + (y - 1 - p)] = x;
    }
}

hipError_t launch_tables(const double* gamma, const double* beta, int64_t n_pl, int32_t R, int32_t cmin,
                         const double* deltas, int64_t pl_per_inst, float2* phase, float2* mix, hipStream_t st) {
    const int64_t total = n_pl * R;
    int64_t blocks = (total + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(k_tables, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, st, gamma, beta, n_pl, R,
                       cmin, deltas, pl_per_inst, phase, mix);
    return hipGetLastError();
}

hipError_t launch_plan_tables(PlanTabs a, int32_t max_k, hipStream_t st) {
    // a workgroup per cone (and layer), more where that leaves the chip idle; a grid holds fewer than 2^32 threads
    const int64_t parts = max_k > 8 ? int64_t{1} << (max_k - 8) : 1, few = 16384 / std::max<int64_t>(a.n_cones, 1);
    a.cut_parts = static_cast<uint32_t>(std::clamp<int64_t>(few, 1, parts));
    a.in_parts = a.n_in < 64 ? 8 : 1;
    const int64_t layers = std::max(a.p - 1, 1), most = (int64_t{UINT32_MAX} / 64 - 16384) / (2 * layers);
    const int64_t n_cones = a.n_cones, n_in = a.n_in;
    for (int64_t c0 = 0; c0 < std::max(n_cones, n_in); c0 += most) {
        PlanTabs q = a;
        q.cones += std::min(c0, n_cones);
        q.in += std::min(c0, n_in);
        q.n_cones = std::clamp<int64_t>(n_cones - c0, 0, most);
        q.n_in = std::clamp<int64_t>(n_in - c0, 0, most);
        const int64_t blocks = q.n_cones * q.cut_parts + q.n_in * layers * q.in_parts;
        hipLaunchKernelGGL(k_plan_tables, dim3(static_cast<unsigned>(blocks)), dim3(64), 0, st, q);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// g[i][l][m] *= delta of m's instance for l < p: per-term gamma derivatives from cut values
// counted in the weight unit to radians (only when the caller asks for the per-term gradient).
__global__ void k_scale_gamma_terms(double* __restrict__ g, int64_t P, int32_t p, int32_t M,
                                    const int64_t* __restrict__ inst_orbit, int32_t n_inst,
                                    const double* __restrict__ deltas) {
    const int64_t total = P * p * static_cast<int64_t>(M);
    for (int64_t t = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; t < total;
         t += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        const int64_t i = t / (static_cast<int64_t>(p) * M);
        const int64_t r = t - i * p * static_cast<int64_t>(M);
        const int64_t m = r % M;
        int32_t lo = 0, hi = n_inst;   // instance j with inst_orbit[j] <= m < inst_orbit[j + 1]
        while (hi - lo > 1) {
            const int32_t mid = (lo + hi) / 2;
            if (inst_orbit[mid] <= m) lo = mid; else hi = mid;
        }
        g[(i * 2 * p) * static_cast<int64_t>(M) + r] *= deltas[lo];
    }
}

hipError_t launch_scale_gamma_terms(double* g, int64_t P, int32_t p, int32_t M, const int64_t* inst_orbit,
                                    int32_t n_inst, const double* deltas, hipStream_t st) {
    const int64_t total = P * p * static_cast<int64_t>(M);
    int64_t blocks = (total + 255) / 256;
    if (blocks > 8192) blocks = 8192;
    if (blocks < 1) return hipSuccess;
    hipLaunchKernelGGL(k_scale_gamma_terms, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, st, g, P, p, M,
                       inst_orbit, n_inst, deltas);
    return hipGetLastError();
}

int64_t combine_chunk(uint32_t ny) { return static_cast<int64_t>(UINT32_MAX) / (256 * static_cast<int64_t>(ny)); }

hipError_t launch_combine(const double* W, const double* Wg, const double* zz, const double* g, int32_t M, int32_t p,
                          const int64_t* inst_orbit, const double* deltas, int32_t n_inst, int64_t Pc,
                          int64_t P_out, int64_t i0, double* energy, double* dgamma, double* dbeta, hipStream_t st) {
    const unsigned ny = (g != nullptr) ? static_cast<unsigned>(1 + 2 * p) : 1u;
    const int64_t nb = static_cast<int64_t>(n_inst) * Pc;
    // a grid holds fewer than 2^32 threads
    if (M <= 64) {
        const int64_t n = nb * ny, CH = static_cast<int64_t>(UINT32_MAX) / 64 / 4 * 4;
        for (int64_t t0 = 0; t0 < n; t0 += CH) {
            const unsigned nx = static_cast<unsigned>((std::min(CH, n - t0) + 3) / 4);
            hipLaunchKernelGGL(k_combine_small, dim3(nx), dim3(256), 0, st, W, Wg, zz, g, M, p, inst_orbit, deltas, Pc, P_out,
                               i0, t0, n, static_cast<int32_t>(ny), energy, dgamma, dbeta);
            const hipError_t e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }
    // one block per (instance, point, value)
    const int64_t CH = combine_chunk(ny);
    for (int64_t b0 = 0; b0 < nb; b0 += CH) {
        const unsigned nx = static_cast<unsigned>(nb - b0 < CH ? nb - b0 : CH);
        hipLaunchKernelGGL(k_combine, dim3(nx, ny), dim3(256), 0, st, W, Wg, zz, g, M, p, inst_orbit, deltas, Pc, P_out,
                           i0, b0, energy, dgamma, dbeta);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace qaoa
