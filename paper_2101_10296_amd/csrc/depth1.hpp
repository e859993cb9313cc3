// Depth-1 terms in closed form: descriptors and launchers (depth1.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

namespace qaoa {

// One depth-1 light cone: the couplings of u and v to each other qubit of the cone.
struct ConeD1 {
    int32_t orbit;   // term index m (output column)
    int32_t inst;    // instance of the cone
    int32_t off;     // first neighbour in D1Args.nb
    int32_t n;       // neighbours (k - 2)
    double wuv;      // coupling of the edge itself (weight units; real weights as they are)
};

struct D1Args {
    const ConeD1* cones;
    const double2* nb;       // (w_ux, w_vx) of every neighbour, 0 = no edge
    int64_t n_cones;
    const double* gamma;     // [inst][gamma_P]
    const double* beta;
    int64_t gamma_P;         // points per instance in gamma and beta
    const double* deltas;    // weight unit of each instance
    int64_t P;               // points of this call
    int32_t M;               // terms (orbits, all instances)
    double* zz;              // [P][M] (k_depth1_point: may be null)
    double* g;               // [P][2][M]: d zz / d theta, d zz / d beta (k_depth1_point: may be null)
    double g_scale;          // k_depth1_point: factor of the stored d zz / d theta (the unit, for radians)
};

constexpr int D1_POINT = 2048;   // orbits of a plan whose terms and sums are one launch

// Items t = point * n_cones + slot, item0 <= t < n_items.
hipError_t launch_depth1_terms(const D1Args& a, int64_t item0, int64_t n_items, bool grad, hipStream_t st);
// One instance, cones[m] of orbit m: terms and weighted sums together.
hipError_t launch_depth1_point(const D1Args& a, const double* W, double* energy, double* dgamma, double* dbeta,
                               hipStream_t st);

}  // namespace qaoa
