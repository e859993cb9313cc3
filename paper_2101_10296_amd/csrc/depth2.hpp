// Depth-2 light cones that are trees: descriptors and launchers (depth2.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace qaoa {

constexpr int D2_TABLE = 32;   // kinds of branches, and of sides, that a workgroup evaluates once for its cones
constexpr int D2_POINT = 256;  // orbits of a plan whose terms and sums are one launch

// A neighbour of u or v (or, without leaves, the edge itself): its coupling and those of its leaves.
struct D2Type {
    double w;
    int32_t leaf, n_leaf;      // entries of D2Args::leaf
};
struct D2Leaf {
    double w;                  // m leaves of coupling w (its sign has no part)
    int32_t m, pad_;
};
// The neighbours of u or of v: their types in D2Args::branch
struct D2SideDef {
    int32_t off, n;
};
struct alignas(16) D2Cone {
    int32_t orbit;
    int32_t edge;              // type of the edge's coupling
    int32_t u, v;              // sides
};

struct D2Args {
    const D2Cone* cones;       // of the launch
    const D2SideDef* sides;
    const int32_t* branch;
    const D2Type* types;
    const D2Leaf* leaf;
    int32_t n_types, n_sides;
    const double* gamma;       // [inst][gamma_P][2]
    const double* beta;
    int64_t gamma_P;
    const double* deltas;
    int32_t P, point0;         // points of the launch
    int32_t M;
    int32_t units;             // cones
    int32_t upw;               // cones per thread
    int32_t blocks;            // workgroups per point
    const int32_t* seg;        // segments of one instance each, as InArgs'
    int32_t n_seg, inst0;
    double* zz;                // [P][M], rows from point 0 of the call
    double* g;                 // [P][4][M]
};

hipError_t launch_depth2(const D2Args& a, bool grad, hipStream_t st);
// terms (zz, g: null where the caller does not ask for them; g in radians) and their weighted sums;
// one instance, cones of all orbits in order, at most D2_POINT
hipError_t launch_depth2_point(const D2Args& a, const double* W, double* energy, double* dgamma, double* dbeta,
                               hipStream_t st);

}  // namespace qaoa
