// Several small classes of inner-state cones (numbers of inner qubits, with and without leaves) in one
// launch.
//
// The classes' launches ran one after the other, the small ones each bound by the latency of one unit,
// and so did the sums of their parts.  Here every workgroup looks up its class and branches to its
// code; a second launch adds the parts of all classes.  Units, sums and their order are those of
// k_inner and k_inner_sum (same bits).  One call on one MI355X: energies of a random 4-regular n = 60,
// p = 2 (7 and 8 inner qubits) 36 -> 29 us; energy and gradient of seven random 3-regular graphs at
// 8 points (cones with cycles of 5 and 6 inner qubits) 50 -> 37 us.
#include "inner_impl.hpp"

namespace qaoa {
namespace {

template <bool GRAD, int PP>
__global__ void __launch_bounds__(256, GRAD && PP == 0 ? 2 : 4) k_inner_mix(InArgs a, InMix m) {
    extern __shared__ __attribute__((aligned(16))) float2 dyn[];   // cosines and phase rows (in_rows); then (PP = 0) sums
    __shared__ CfgIn cfg_all[4][64];
    __shared__ InShared sh;
    __shared__ double2 s_z[4][16];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int p = PP ? PP : a.p, R = a.R;
    const int point = blockIdx.x / m.blocks + a.point0;
    const int blk = blockIdx.x % m.blocks;
    int ci = 0;
    while (ci + 1 < m.n && m.c[ci + 1].block0 <= blk) ++ci;
    const InMix::Class& c = m.c[ci];
    a.units = c.units;
    a.n_seg = c.n_seg;
    a.seg = c.seg;
    a.inst0 = c.inst0;
    int u0, u1, inst;
    in_segment(a, blk - c.block0, 4, u0, u1, inst);
    in_rows(a, p, inst, point, tid, 256, dyn, sh);
    __syncthreads();
    const int u = u0 + wave;
    if (u >= u1) return;
    double* lsum = nullptr;   // PP = 0: [2p + 1][64] sums of this wave's lanes
    if constexpr (PP == 0) lsum = reinterpret_cast<double*>(in_phase(a, dyn) + (3 + p) * R + ((3 + p) * R & 1)) + wave * (2 * p + 1) * 64;
    const int nv = GRAD ? 2 * p + 1 : 1, chunks = c.chunks;
    const int slot = u / chunks, ch = u - slot * chunks;
    const ConeIn& cd = a.cones[c.cone0 + slot];
    double* out = chunks > 1 || m.all ? a.part + c.part0 + (static_cast<size_t>(point - a.point0) * c.units + u) * nv : nullptr;
    auto put = [&](int code, double x) {
        if (out) out[code] = x;
        else if (code == 0) a.zz[static_cast<size_t>(point) * a.M + cd.orbit] = x;
        else a.g[(static_cast<size_t>(point) * 2 * p + (code - 1)) * a.M + cd.orbit] = x;
    };
    auto run = [&](auto K) {
        constexpr int KIN = decltype(K)::value;
        if constexpr (KIN >= 4 || PP == 2) {
            const InLane<KIN> ln(lane);
            if (c.signs) in_unit<KIN, GRAD, PP, false, true>(a, cd, ch, chunks, lane, ln, dyn, sh, cfg_all[wave], s_z[wave], lsum, put);
            else in_unit<KIN, GRAD, PP, false, false>(a, cd, ch, chunks, lane, ln, dyn, sh, cfg_all[wave], s_z[wave], lsum, put);
        }
    };
    switch (c.kin) {
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

}  // namespace

hipError_t launch_inner_mix(const InArgs& a, const InMix& m, bool grad, hipStream_t st) {
    const int64_t blocks = static_cast<int64_t>(m.blocks) * a.P;
    if (m.n < 1 || m.n > IN_CLASSES || a.p < 2 || a.p > IN_PMAX) return hipErrorInvalidValue;
    if (blocks <= 0) return hipSuccess;
    size_t lds = in_rows_bytes(a);
    if (a.p > 2 && grad) lds += 8 + 4 * static_cast<size_t>(2 * a.p + 1) * 64 * sizeof(double);
    const dim3 grid(static_cast<unsigned>(blocks)), block(256);
    if (a.p == 2) {
        if (grad) hipLaunchKernelGGL((k_inner_mix<true, 2>), grid, block, lds, st, a, m);
        else hipLaunchKernelGGL((k_inner_mix<false, 2>), grid, block, lds, st, a, m);
    } else {
        if (grad) hipLaunchKernelGGL((k_inner_mix<true, 0>), grid, block, lds, st, a, m);
        else hipLaunchKernelGGL((k_inner_mix<false, 0>), grid, block, lds, st, a, m);
    }
    return hipGetLastError();
}

}  // namespace qaoa
