// Small plans of light cones on their inner qubits: every term of a point and their weighted sums
// in one launch.
//
// A plan that symmetry reduces to a few cones has a few waves of work per point, and a call is
// bound by its launches: one per number of inner qubits, the sum of a cone's parts, and the
// weighted sums.  Here a workgroup takes one point, a wave each unit of work (a cone's
// configurations or a part of them, any number of inner qubits), and the sums follow in the same
// workgroup, in the order of k_inner_sum and k_combine: results are the same bit for bit, and
// no term goes through device memory.
//
// Bound: the serial chain of one unit (phase rows, descriptors and tables through L2, then about
// 2000 instructions of one wave).  Energy and gradient of C_10000(1,2) at p = 2 (inner states of
// 6 and 7 qubits, one unit each), one point: 18.8 us a call in three launches, 13.6 in one (now 9.7,
// with the set-up on three waves and less host time around the call).
#include "depth2_impl.hpp"
#include "inner_impl.hpp"

namespace qaoa {
namespace {

// Value y of the weighted sums: the tree of k_combine over the terms in orbit order (its threads beyond
// the last orbit hold zeros).
template <class Q>
__device__ __forceinline__ void in_point_sums(const InArgs& a, const Q& q, int y, int point, int p, double delta,
                                              const double (&s_term)[IN_POINT][2 * IN_PMAX + 1]) {
    double t[IN_POINT];
#pragma unroll
    for (int m = 0; m < IN_POINT; ++m) {
        t[m] = 0.0;
        if (m < a.M) t[m] = y == 0 ? q.W[m] * (1.0 - s_term[m][y]) * 0.5 : -0.5 * q.W[m] * s_term[m][y];
    }
#pragma unroll
    for (int s = IN_POINT / 2; s > 0; s >>= 1)
#pragma unroll
        for (int m = 0; m < s; ++m) t[m] += t[m + s];
    if (y == 0) q.energy[point] = t[0];
    else if (y <= p) q.dgamma[static_cast<size_t>(point) * p + (y - 1)] = a.g ? t[0] : delta * t[0];
    else q.dbeta[static_cast<size_t>(point) * p + (y - 1 - p)] = t[0];
}

template <bool GRAD, int PP>
__global__ void __launch_bounds__(64 * in_point_waves(GRAD, PP), GRAD && PP == 0 ? 2 : 4)
k_inner_point(InArgs a, D2Args d, InPoint q) {
    extern __shared__ __attribute__((aligned(16))) float2 dyn[];   // cosines and phase rows; then (PP = 0) sums
    __shared__ InShared sh;
    __shared__ double2 s_z[in_point_waves(GRAD, PP)][16];
    __shared__ double s_val[IN_POINT][2 * IN_PMAX + 1];    // parts of cones
    __shared__ double s_term[IN_POINT][2 * IN_PMAX + 1];   // orbits
    const int tid = threadIdx.x, lane = tid & 63, waves = blockDim.x >> 6;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int p = PP ? PP : a.p, R = a.R;
    const int nv = GRAD ? 2 * p + 1 : 1;
    const int point = blockIdx.x + a.point0;
    in_rows(a, p, 0, point, tid, blockDim.x, dyn, sh);
    __syncthreads();
    double* lsum = nullptr;
    if constexpr (PP == 0) lsum = reinterpret_cast<double*>(in_phase(a, dyn) + (3 + p) * R + ((3 + p) * R & 1)) + wave * (2 * p + 1) * 64;
    for (int u = wave; u < q.n; u += waves) {
        const InPoint::Unit un = q.unit[u];
        if constexpr (PP == 2) {
            if (un.trees) {
                if (lane < un.trees) {
                    const double delta = a.deltas[0];
                    const size_t ip = static_cast<size_t>(point) * 2;
                    double v[5];
                    d2_cone<GRAD>(d, d.cones[un.cone + lane], a.gamma[ip] * delta, a.gamma[ip + 1] * delta,
                                  d2_angles(a.beta[ip], a.beta[ip + 1]), v);
                    for (int i = 0; i < nv; ++i) s_val[un.part + lane][i] = v[i];
                }
                continue;
            }
        }
        const ConeIn& cd = a.cones[un.cone];
        auto run = [&](auto K) {
            constexpr int KIN = decltype(K)::value;
            if constexpr (KIN >= 4 || PP == 2) {
                const InLane<KIN> ln(lane);
                in_unit<KIN, GRAD, PP, true, true>(a, cd, un.chunk, un.chunks, lane, ln, dyn, sh, nullptr, s_z[wave], lsum,
                                             [&](int code, double x) { s_val[un.part][code] = x; });
            }
        };
        switch (un.kin) {
            case 3: run(std::integral_constant<int, 3>{}); break;
            case 4: run(std::integral_constant<int, 4>{}); break;
            case 5: run(std::integral_constant<int, 5>{}); break;
            case 6: run(std::integral_constant<int, 6>{}); break;
            case 7: run(std::integral_constant<int, 7>{}); break;
            case 8: run(std::integral_constant<int, 8>{}); break;
            case 9: run(std::integral_constant<int, 9>{}); break;
            default: run(std::integral_constant<int, 10>{}); break;
        }
    }
    __syncthreads();
    if (tid >= nv) return;
    // thread y: the terms' value y
    const int y = tid;
    const double delta = a.deltas[0];
    const double gs = y >= 1 && y <= p && a.g ? delta : 1.0;   // the caller's terms are in radians
    for (int u = 0; u < q.n_part;) {
        const InPoint::Part pt = q.part[u];
        double x = 0.0;
        for (int c = 0; c < pt.chunks; ++c) x += s_val[u + c][y];
        u += pt.chunks;
        x *= gs;
        const int m = pt.orbit;
        s_term[m][y] = x;
        if (y == 0) {
            if (a.zz) a.zz[static_cast<size_t>(point) * a.M + m] = x;
        } else if (a.g) {
            a.g[(static_cast<size_t>(point) * 2 * p + (y - 1)) * a.M + m] = x;
        }
    }
    in_point_sums(a, q, y, point, p, delta, s_term);
}

// One workgroup per point: a thread per (cone, value) adds the cone's parts as k_inner_sum, then the
// sums.  Bound by its launch: the 18-qubit cone of a torus, 19 parts, 32 points, the whole call 19.2 us
// with the parts, the terms and the sums in launches of their own, 17.5 here.
template <bool GRAD>
__global__ void __launch_bounds__(320) k_inner_point_sum(InArgs a, InPointSum q) {
    __shared__ double s_term[IN_POINT][2 * IN_PMAX + 1];
    const int tid = threadIdx.x, p = a.p, nv = GRAD ? 2 * p + 1 : 1;
    const int point = blockIdx.x + a.point0;
    const double delta = a.deltas[0];
    if (tid < q.n * nv) {
        const int i = tid / nv, v = tid - i * nv;
        const InPointSum::Cone& c = q.c[i];
        const double* src = a.part + c.part0 + (static_cast<size_t>(blockIdx.x) * c.units + c.unit0) * nv + v;
        double x = in_part_sum(src, c.chunks, nv);
        if (v >= 1 && v <= p && a.g) x *= delta;   // the caller's terms are in radians
        s_term[c.orbit][v] = x;
        if (v == 0) {
            if (a.zz) a.zz[static_cast<size_t>(point) * a.M + c.orbit] = x;
        } else if (a.g) {
            a.g[(static_cast<size_t>(point) * 2 * p + (v - 1)) * a.M + c.orbit] = x;
        }
    }
    __syncthreads();
    if (tid < nv) in_point_sums(a, q, tid, point, p, delta, s_term);
}

}  // namespace

hipError_t launch_inner_point_sum(const InArgs& a, const InPointSum& q, bool grad, hipStream_t st) {
    if (q.n < 1 || q.n > IN_POINT || a.M != q.n || a.p < 2 || a.p > IN_PMAX) return hipErrorInvalidValue;
    if (a.P <= 0) return hipSuccess;
    const dim3 grid(static_cast<unsigned>(a.P)), block(320);
    if (grad) hipLaunchKernelGGL(k_inner_point_sum<true>, grid, block, 0, st, a, q);
    else hipLaunchKernelGGL(k_inner_point_sum<false>, grid, block, 0, st, a, q);
    return hipGetLastError();
}

hipError_t launch_inner_point(const InArgs& a0, const D2Args& d, const InPoint& q, bool grad, int64_t n_points, hipStream_t st) {
    if (q.n < 1 || q.n > IN_POINT || q.n_part > IN_POINT || a0.M > IN_POINT || a0.p < 2 || a0.p > IN_PMAX) return hipErrorInvalidValue;
    const bool sums = a0.p > 2 && grad;
    // three waves at least where points leave compute units idle: the set-up's chains (in_rows) side by side
    const int waves = std::max(n_points <= 256 ? 3 : 1, std::min<int>(q.n, in_point_waves(grad, a0.p == 2 ? 2 : 0)));
    size_t lds = in_rows_bytes(a0);
    if (sums) lds += 8 + static_cast<size_t>(waves) * (2 * a0.p + 1) * 64 * sizeof(double);
    // a grid holds fewer than 2^32 threads
    const int64_t CH = static_cast<int64_t>(UINT32_MAX) / (64 * waves);
    for (int64_t p0 = 0; p0 < n_points; p0 += CH) {
        InArgs a = a0;
        a.point0 = static_cast<int32_t>(p0);
        const dim3 grid(static_cast<unsigned>(std::min(CH, n_points - p0))), block(64 * waves);
        if (a.p == 2) {
            if (grad) hipLaunchKernelGGL((k_inner_point<true, 2>), grid, block, lds, st, a, d, q);
            else hipLaunchKernelGGL((k_inner_point<false, 2>), grid, block, lds, st, a, d, q);
        } else {
            if (grad) hipLaunchKernelGGL((k_inner_point<true, 0>), grid, block, lds, st, a, d, q);
            else hipLaunchKernelGGL((k_inner_point<false, 0>), grid, block, lds, st, a, d, q);
        }
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace qaoa
