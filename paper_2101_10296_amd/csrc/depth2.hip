// Kernels of the depth-2 closed form (depth2_impl.hpp).
//
// Where the plan has few kinds of sides (unit and small integer weights), a workgroup evaluates each
// kind of branch and of side once, in LDS, and a term is some 130 FP64 operations on two sides and
// an edge: bound by the writes of the terms (n = 10000, random 3-regular, 256 points, energy and
// gradient: 154 MB in 36 us, 4.3 TB/s; 112 us where each term multiplied its own branches).
// Otherwise (real weights: every branch its own kind) a term takes some 20 sines and cosines: bound
// by FP64 issue.
//
// Calls on one MI355X, energy and gradient at p = 2: that graph 215.6 ms on the kernels for whole
// cones, 2.32 ms as states of the inner qubits, 0.136 ms here (90 us of it the weighted sums and the
// 65 cones with cycles); Gaussian weights, n = 104, 19 points, 390 -> 87 us (most of it the cones
// with cycles); a ring at 16384 points 118 -> 51 (states, one launch) -> 6.7 us.
#include "depth2_impl.hpp"

namespace qaoa {
namespace {

// One thread per cone, upw of them 256 apart: neighbouring threads write neighbouring orbits.
template <bool GRAD, bool TABLE>
__global__ void __launch_bounds__(256) k_depth2(D2Args a) {
    __shared__ D2Val s_v[TABLE ? D2_TABLE : 1];
    __shared__ D2Side<GRAD> s_s[TABLE ? D2_TABLE : 1];
    __shared__ D2Angles s_a;
    const int tid = threadIdx.x;
    const int64_t point = blockIdx.x / a.blocks + a.point0;
    const int blk = blockIdx.x % a.blocks, per = 256 * a.upw;
    int u0 = blk * per, u1 = a.units, inst = a.inst0;
    if (a.n_seg > 1) {   // the segment of one instance that holds this workgroup
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
    const size_t ip = (static_cast<size_t>(inst) * a.gamma_P + point) * 2;
    const double t1 = a.gamma[ip] * a.deltas[inst], t2 = a.gamma[ip + 1] * a.deltas[inst];
    if (tid == 255) s_a = d2_angles(a.beta[ip], a.beta[ip + 1]);
    if constexpr (TABLE)
        if (tid < a.n_types) s_v[tid] = d2_val(a.types[tid], a.leaf, t1, t2);
    __syncthreads();
    const D2Angles an = s_a;
    if constexpr (TABLE) {
        if (tid < a.n_sides) {
            const D2SideDef d = a.sides[tid];
            s_s[tid] = d2_side<GRAD>(d.n, an, [&](int i) { return s_v[a.branch[d.off + i]]; });
        }
        __syncthreads();
    }
    for (int u = u0 + tid, i = 0; i < a.upw && u < u1; ++i, u += 256) {
        const D2Cone c = a.cones[u];
        double v[5];
        if constexpr (TABLE) d2_term<GRAD>(s_v[c.edge], s_s[c.u], s_s[c.v], an, v);
        else d2_cone<GRAD>(a, c, t1, t2, an, v);
        a.zz[static_cast<size_t>(point) * a.M + c.orbit] = v[0];
        if constexpr (GRAD) {
#pragma unroll
            for (int j = 0; j < 4; ++j) a.g[(static_cast<size_t>(point) * 4 + j) * a.M + c.orbit] = v[1 + j];
        }
    }
}

// Terms and their orbit-weighted sums in one launch where every cone is a tree, up to 256 orbits (one
// per thread of a point's lanes; beyond, a thread per term fills the chip better): 2^lb lanes per point, an orbit each, then the tree
// of k_combine (whose threads beyond the last orbit hold zeros).
template <bool GRAD>
__global__ void __launch_bounds__(256)
k_depth2_point(D2Args a, int lb, const double* __restrict__ W, double* __restrict__ energy, double* __restrict__ dgamma,
               double* __restrict__ dbeta) {
    constexpr int NV = GRAD ? 5 : 1;
    __shared__ double sh[NV][256];
    const int lanes = 1 << lb, lane = threadIdx.x & (lanes - 1);
    const int64_t point = blockIdx.x * static_cast<int64_t>(256 >> lb) + (threadIdx.x >> lb);
    const double delta = a.deltas[0];
    const double gs = a.g ? delta : 1.0;   // the caller's terms are in radians
    double acc[5] = {};
    if (point < a.P && lane < a.units) {
        const double t1 = a.gamma[point * 2] * delta, t2 = a.gamma[point * 2 + 1] * delta;
        double v[5];
        d2_cone<GRAD>(a, a.cones[lane], t1, t2, d2_angles(a.beta[point * 2], a.beta[point * 2 + 1]), v);
        if (a.zz) a.zz[static_cast<size_t>(point) * a.M + lane] = v[0];
        const double w = W[lane];
        acc[0] = w * (1.0 - v[0]) * 0.5;
        if constexpr (GRAD) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const double x = j < 2 ? v[1 + j] * gs : v[1 + j];
                if (a.g) a.g[(static_cast<size_t>(point) * 4 + j) * a.M + lane] = x;
                acc[1 + j] = -0.5 * w * x;
            }
        }
    }
#pragma unroll
    for (int i = 0; i < NV; ++i) sh[i][threadIdx.x] = acc[i];
    for (int s = lanes >> 1; s > 0; s >>= 1) {
        __syncthreads();
        if (lane < s) {
#pragma unroll
            for (int i = 0; i < NV; ++i) sh[i][threadIdx.x] += sh[i][threadIdx.x + s];
        }
    }
    if (lane == 0 && point < a.P) {
        energy[point] = sh[0][threadIdx.x];
        if constexpr (GRAD) {
            const double d = a.g ? 1.0 : delta;
            dgamma[point * 2] = d * sh[1][threadIdx.x];
            dgamma[point * 2 + 1] = d * sh[2][threadIdx.x];
            dbeta[point * 2] = sh[3][threadIdx.x];
            dbeta[point * 2 + 1] = sh[4][threadIdx.x];
        }
    }
}

}  // namespace

hipError_t launch_depth2(const D2Args& a, bool grad, hipStream_t st) {
    const int64_t blocks = static_cast<int64_t>(a.blocks) * a.P;
    if (blocks <= 0) return hipSuccess;
    const dim3 grid(static_cast<unsigned>(blocks)), block(256);
    if (a.n_types <= D2_TABLE && a.n_sides <= D2_TABLE) {
        if (grad) hipLaunchKernelGGL((k_depth2<true, true>), grid, block, 0, st, a);
        else hipLaunchKernelGGL((k_depth2<false, true>), grid, block, 0, st, a);
    } else {
        if (grad) hipLaunchKernelGGL((k_depth2<true, false>), grid, block, 0, st, a);
        else hipLaunchKernelGGL((k_depth2<false, false>), grid, block, 0, st, a);
    }
    return hipGetLastError();
}

hipError_t launch_depth2_point(const D2Args& a, const double* W, double* energy, double* dgamma, double* dbeta,
                               hipStream_t st) {
    if (a.units < 1 || a.units > D2_POINT || a.units != a.M) return hipErrorInvalidValue;
    int lb = 0;
    while ((1 << lb) < a.units) ++lb;
    const int64_t per = 256 >> lb, blocks = (a.P + per - 1) / per;
    // a grid holds fewer than 2^32 threads
    constexpr int64_t CH = static_cast<int64_t>(UINT32_MAX) / 256;
    for (int64_t b0 = 0; b0 < blocks; b0 += CH) {
        D2Args c = a;
        const int64_t p0 = b0 * per;
        c.P = static_cast<int32_t>(a.P - p0);
        c.gamma = a.gamma + p0 * 2;
        c.beta = a.beta + p0 * 2;
        c.zz = a.zz ? a.zz + static_cast<size_t>(p0) * a.M : nullptr;
        c.g = a.g ? a.g + static_cast<size_t>(p0) * 4 * a.M : nullptr;
        const dim3 grid(static_cast<unsigned>(std::min<int64_t>(CH, blocks - b0)));
        if (dgamma)
            hipLaunchKernelGGL(k_depth2_point<true>, grid, dim3(256), 0, st, c, lb, W, energy + p0, dgamma + p0 * 2,
                               dbeta + p0 * 2);
        else
            hipLaunchKernelGGL(k_depth2_point<false>, grid, dim3(256), 0, st, c, lb, W, energy + p0, nullptr, nullptr);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace qaoa
