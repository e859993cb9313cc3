// Kernels of inner_tree_impl.hpp.
#include "inner_tree_impl.hpp"

namespace qaoa {
namespace {

template <int KIN, bool GRAD>
__global__ void __launch_bounds__(256, 4) k_inner_tree(InArgs a) {
    extern __shared__ __attribute__((aligned(16))) float2 dyn[];   // cosines and phase rows (in_rows)
    __shared__ InShared sh;
    __shared__ double2 s_typ[TR_TYPES];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int point = blockIdx.x / a.blocks + a.point0;
    int u0, u1, inst;
    in_segment(a, blockIdx.x % a.blocks, 16 * a.upw, u0, u1, inst);
    in_rows(a, 2, inst, point, tid, 256, dyn, sh);
    __syncthreads();
    tr_types(a, tid, 256, dyn, s_typ);
    __syncthreads();
    const InLane<KIN - 1> ln(lane);
    for (int i = 0; i < a.upw; ++i) {
        const int first = u0 + 4 * (wave * a.upw + i);
        if (first >= u1) break;
        const int u = first + (lane >> 4);
        tr_row<KIN, GRAD>(a, a.tr + min(u, u1 - 1), u < u1, lane, ln, dyn, s_typ, sh, [&](int orbit, int code, double x) {
            if (code == 0) a.zz[static_cast<size_t>(point) * a.M + orbit] = x;
            else a.g[(static_cast<size_t>(point) * 4 + (code - 1)) * a.M + orbit] = x;
        });
    }
}

template <int KIN>
void launch(bool grad, const InArgs& a, hipStream_t st) {
    const dim3 grid(static_cast<unsigned>(static_cast<int64_t>(a.blocks) * a.P)), block(256);
    const size_t lds = in_rows_bytes(a);
    if (grad) hipLaunchKernelGGL((k_inner_tree<KIN, true>), grid, block, lds, st, a);
    else hipLaunchKernelGGL((k_inner_tree<KIN, false>), grid, block, lds, st, a);
}

}  // namespace

hipError_t launch_inner_tree(int kin, bool grad, const InArgs& a, hipStream_t st) {
    if (a.p != 2 || a.n_types < 1 || a.n_types > TR_TYPES || a.chunks != 1) return hipErrorInvalidValue;
    if (static_cast<int64_t>(a.blocks) * a.P <= 0) return hipSuccess;
    switch (kin) {
        case 4: launch<4>(grad, a, st); break;
        case 5: launch<5>(grad, a, st); break;
        case 6: launch<6>(grad, a, st); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace qaoa
