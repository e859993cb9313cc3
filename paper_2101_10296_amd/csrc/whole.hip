// Observable tables and dispatch of the shared-state kernel (whole_impl.hpp).
#include "whole_impl.hpp"

namespace qaoa {

hipError_t launch_whole_k5_10(int, bool, const WhArgs&, hipStream_t);
hipError_t launch_whole_k11_14(int, bool, const WhArgs&, hipStream_t);

hipError_t launch_whole(int K, bool grad, const WhArgs& a, hipStream_t st) {
    if (K < WH_KMIN || K > WH_KMAX || a.p < 2) return hipErrorInvalidValue;
    return K <= 10 ? launch_whole_k5_10(K, grad, a, st) : launch_whole_k11_14(K, grad, a, st);
}

namespace {
template <int K>
bool fits(int p, int rowcap, bool realw) {
    return 2 * Wz<K>::IPW * Wz<K>::NPAD * sizeof(float2) + 64 + whole_dyn<K>(p, rowcap, realw) <= 160 * 1024;
}

__global__ void __launch_bounds__(256)
k_whole_obs(const GroupWh* __restrict__ groups, const MemWh* __restrict__ mem, uint32_t n, double* __restrict__ obs) {
    const GroupWh& g = groups[blockIdx.x];
    for (uint32_t x = threadIdx.x; x < n; x += 256) {
        double v = 0.0;
        for (int m = 0; m < g.n_mem; ++m) {
            const MemWh& e = mem[g.mem_off + m];
            v += (((x >> e.u) ^ (x >> e.v)) & 1u) ? 0.5 * e.W : -0.5 * e.W;
        }
        obs[g.v_off + x] = v;
    }
}
}  // namespace

bool whole_fits(int K, int p, int rowcap, bool realw) {
    switch (K) {
        case 5: return fits<5>(p, rowcap, realw);
        case 6: return fits<6>(p, rowcap, realw);
        case 7: return fits<7>(p, rowcap, realw);
        case 8: return fits<8>(p, rowcap, realw);
        case 9: return fits<9>(p, rowcap, realw);
        case 10: return fits<10>(p, rowcap, realw);
        case 11: return fits<11>(p, rowcap, realw);
        case 12: return fits<12>(p, rowcap, realw);
        case 13: return fits<13>(p, rowcap, realw);
        case 14: return fits<14>(p, rowcap, realw);
        default: return false;
    }
}

hipError_t launch_whole_obs(const GroupWh* groups, int64_t n_groups, const MemWh* mem, int K, double* obs, hipStream_t st) {
    if (n_groups <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_whole_obs, dim3(static_cast<unsigned>(n_groups)), dim3(256), 0, st, groups, mem,
                       1u << (K - 1), obs);
    return hipGetLastError();
}

}  // namespace qaoa
