// Shell qubits that couple to one inner qubit only: the average over them is a dephasing of that qubit.
//
// With t = gamma_1 delta and couplings w_j, the mean over the 2^m states of the leaves multiplies the
// density matrix element between x and x' by f = prod_j cos(t w_j) where the qubit's bit differs:
// the channel rho -> (1 + f) / 2 rho + (1 - f) / 2 Z rho Z.  Two signs stand for the leaves' states,
// whatever their number and couplings, and their weights alone depend on the angle: with df = df/dt
// the gradient of gamma_1 gains sum (d weight) <ZZ> over the signs.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "shell_limits.hpp"

namespace qaoa {

// The leaves of one inner qubit: m[i] of coupling +-w[i] (0: none)
struct alignas(16) ZLeaf {
    int16_t w[ZL_W];
    int16_t m[ZL_W];
};

// f and df of one inner qubit; ct[j]: cosine and sine of j t.
__host__ __device__ __forceinline__ double2 z_factor(const ZLeaf& q, const double2* ct) {
    double f = 1.0, df = 0.0;
    for (int i = 0; i < ZL_W && q.m[i]; ++i) {
        const double2 c = ct[q.w[i]];
        for (int j = 0; j < q.m[i]; ++j) {
            df = df * c.x - f * (static_cast<double>(q.w[i]) * c.y);
            f *= c.x;
        }
    }
    return make_double2(f, df);
}

// fac[lane] of the inner qubits in zmask, a lane each.  The others have no factor, and where zmask is 0
// no record stands at z_off: neither is read.
__host__ __device__ __forceinline__ void z_factors(uint32_t zmask, const ZLeaf* leaf, int32_t z_off, const double2* ct, int lane,
                                                   double2* fac) {
    if (lane < 16 && ((zmask >> lane) & 1u)) fac[lane] = z_factor(leaf[z_off + lane], ct);
}

// Weight w of a configuration with the signs z of the qubits zmask, and its derivative.
__host__ __device__ __forceinline__ double z_weight(uint32_t zmask, uint32_t z, const double2* fac, double& w) {
    double dw = 0.0;
    for (; zmask; zmask &= zmask - 1) {
        const int a = __builtin_ctz(zmask);
        const double2 f = fac[a];
        const double s = (z >> a) & 1u ? -0.5 : 0.5;
        const double v = fma(s, f.x, 0.5);
        dw = dw * v + w * (s * f.y);
        w *= v;
    }
    return dw;
}

}  // namespace qaoa
