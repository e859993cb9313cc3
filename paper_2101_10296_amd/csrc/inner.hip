// Tables, chunk sums and dispatch of the inner-state kernel (inner_impl.hpp).
#include "inner.hpp"

namespace qaoa {

hipError_t launch_inner_k3_6(int, bool, const InArgs&, hipStream_t);
hipError_t launch_inner_k7_8(int, bool, const InArgs&, hipStream_t);
hipError_t launch_inner_k9_10(int, bool, const InArgs&, hipStream_t);

hipError_t launch_inner(int kin, bool grad, const InArgs& a, hipStream_t st) {
    if (a.p < 2 || a.p > IN_PMAX || kin < IN_KMIN || kin > IN_KMAX) return hipErrorInvalidValue;
    if (kin <= 6) return launch_inner_k3_6(kin, grad, a, st);
    if (kin <= 8) return launch_inner_k7_8(kin, grad, a, st);
    return launch_inner_k9_10(kin, grad, a, st);
}

namespace {

// The chunks of item t = (point, cone, value), in order.
__device__ __forceinline__ void in_add_parts(const InArgs& a, int64_t t, int32_t n_cones, int32_t nv) {
    const int v = static_cast<int>(t % nv);
    const int64_t pc = t / nv;
    const int32_t c = static_cast<int32_t>(pc % n_cones);
    const int64_t i = pc / n_cones;
    const double* src = a.part + (i * a.units + static_cast<int64_t>(c) * a.chunks) * nv + v;
    const double x = in_part_sum(src, a.chunks, nv);
    const int32_t orbit = a.cones[c].orbit;
    const size_t pt = static_cast<size_t>(i + a.point0);
    if (v == 0) a.zz[pt * a.M + orbit] = x;
    else a.g[(pt * 2 * a.p + (v - 1)) * a.M + orbit] = x;
}

// One thread per (point, cone, value): the chunks of a cone in order.  Bound by the latency of its loads:
// 19 parts of a torus cone at 32 points 6.4 us one load after the other, 4.4 with eight in flight.
__global__ void __launch_bounds__(256) k_inner_sum(InArgs a, int32_t n_cones, int32_t nv) {
    const int64_t n = static_cast<int64_t>(a.P) * n_cones * nv;
    for (int64_t t = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; t < n;
         t += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        in_add_parts(a, t, n_cones, nv);
    }
}

// The same over the classes of k_inner_mix.
__global__ void __launch_bounds__(256) k_inner_mix_sum(InArgs a, InMix m, int32_t nv) {
    for (int64_t t = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; t < m.items;
         t += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        int ci = 0;   // the last class that starts at or before t (those without parts hold no items)
        while (ci + 1 < m.n && m.c[ci + 1].item0 <= t) ++ci;
        const InMix::Class& c = m.c[ci];
        InArgs b = a;
        b.cones = a.cones + c.cone0;
        b.units = c.units;
        b.chunks = c.chunks;
        b.part = a.part + c.part0;
        in_add_parts(b, t - c.item0, c.n_cones, nv);
    }
}

}  // namespace

hipError_t launch_inner_mix_sum(const InArgs& a, const InMix& m, bool grad, hipStream_t st) {
    if (m.items <= 0) return hipSuccess;
    const int64_t blocks = (m.items + 255) / 256;
    hipLaunchKernelGGL(k_inner_mix_sum, dim3(static_cast<unsigned>(blocks < 65536 ? blocks : 65536)), dim3(256), 0, st, a,
                       m, grad ? 2 * a.p + 1 : 1);
    return hipGetLastError();
}

hipError_t launch_inner_sum(const InArgs& a, int32_t n_cones, bool grad, hipStream_t st) {
    const int nv = grad ? 2 * a.p + 1 : 1;
    const int64_t n = static_cast<int64_t>(a.P) * n_cones * nv;
    if (n <= 0) return hipSuccess;
    const int64_t blocks = (n + 255) / 256;
    hipLaunchKernelGGL(k_inner_sum, dim3(static_cast<unsigned>(blocks < 65536 ? blocks : 65536)), dim3(256), 0, st, a,
                       n_cones, nv);
    return hipGetLastError();
}

}  // namespace qaoa
