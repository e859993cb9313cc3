// Tables, sums and instantiations of the workgroup kernel of inner states (wide_impl.hpp).
#include "wide_impl.hpp"

namespace qaoa {

hipError_t launch_wide(int kin, bool grad, const WdArgs& a, hipStream_t st) {
    if (a.p < 2 || a.p > WD_PMAX) return hipErrorInvalidValue;
    switch (kin) {
        case 11: return launch_wide_k<11>(grad, a, st);
        case 12: return launch_wide_k<12>(grad, a, st);
        case 13: return launch_wide_k<13>(grad, a, st);
        case 14: return launch_wide_k<14>(grad, a, st);
        default: return hipErrorInvalidValue;
    }
}

namespace {

__global__ void __launch_bounds__(256)
k_wide_tables(const ConeWd* __restrict__ cones, const int32_t* __restrict__ ea, const int32_t* __restrict__ eb,
              const int32_t* __restrict__ ew, int32_t p, uint8_t* __restrict__ tab) {
    const ConeWd& cd = cones[blockIdx.x];
    const uint32_t n = 1u << cd.kin;
    const int l = 2 + blockIdx.y;
    uint8_t* out = tab + cd.tab_off + static_cast<size_t>(l - 2) * n;
    const int m = cd.mixed[l - 1], cmin = cd.base[l] + cd.cut_min;
    for (uint32_t x = blockIdx.z * 256 + threadIdx.x; x < n; x += gridDim.z * 256) {
        int32_t c = 0;
        for (int32_t e = 0; e < cd.n_edges; ++e) {
            const int32_t i = ea[cd.edge_off + e], j = eb[cd.edge_off + e];
            if (j < m) c += ew[cd.edge_off + e] * static_cast<int32_t>(((x >> i) ^ (x >> j)) & 1u);
        }
        out[x] = static_cast<uint8_t>(c - cmin);
    }
}

// One workgroup per (cone, point): the units of the cone, a fixed number of lanes per value.
__global__ void __launch_bounds__(256) k_wide_sum(WdArgs a, int32_t n_cones, int32_t nv) {
    __shared__ double sh[256];
    const int64_t b = blockIdx.x;
    const int32_t c = static_cast<int32_t>(b % n_cones);
    const int64_t pt = b / n_cones;
    const ConeWd& cd = a.cones[a.cone0 + c];
    const int v = threadIdx.x & 7, q = threadIdx.x >> 3;   // at most 7 values
    double x = 0.0;
    if (v < nv) {
        const double* src = a.part + (pt * a.all_units + (cd.first_unit - a.sum_unit0)) * nv + v;
        for (int u = q; u < cd.n_units; u += 32) x += src[static_cast<size_t>(u) * nv];
    }
    sh[threadIdx.x] = x;
    for (int s = 128; s >= 8; s >>= 1) {
        __syncthreads();
        if (static_cast<int>(threadIdx.x) < s) sh[threadIdx.x] += sh[threadIdx.x + s];
    }
    if (threadIdx.x < 8 && v < nv) {
        const size_t point = static_cast<size_t>(pt + a.point0);
        if (v == 0) a.zz[point * a.M + cd.orbit] = sh[threadIdx.x];
        else a.g[(point * 2 * a.p + (v - 1)) * a.M + cd.orbit] = sh[threadIdx.x];
    }
}

}  // namespace

hipError_t launch_wide_sum(const WdArgs& a, int32_t n_cones, bool grad, hipStream_t st) {
    const int64_t blocks = static_cast<int64_t>(n_cones) * a.P;
    if (blocks <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_wide_sum, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, st, a, n_cones,
                       grad ? 2 * a.p + 1 : 1);
    return hipGetLastError();
}

hipError_t launch_wide_tables(const ConeWd* cones, int64_t n_cones, const int32_t* ea, const int32_t* eb,
                              const int32_t* ew, int32_t p, uint8_t* tab, hipStream_t st) {
    if (n_cones <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_wide_tables, dim3(static_cast<unsigned>(n_cones), static_cast<unsigned>(p - 1), n_cones < 64 ? 8 : 1), dim3(256), 0,
                       st, cones, ea, eb, ew, p, tab);
    return hipGetLastError();
}

}  // namespace qaoa
