// Groups of light cones with the same qubits: descriptors and launchers (whole.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace qaoa {

constexpr int WH_KMIN = 5;      // cone qubits
constexpr int WH_KMAX = 14;
constexpr int WH_MEMBERS = 3;   // terms that make a group

struct GroupWh {
    int32_t inst;
    int32_t rep;                // column that carries the group's gradient
    int32_t mem_off, n_mem;     // members
    int64_t cut_off;            // cut table of the representative cone (bytes; real weights: floats)
    int64_t v_off;              // observable table (doubles)
    double scale;               // its unit: the largest power of two up to the members' largest weight
    int32_t cut_row;            // phase row index of table value 0: cut_min of the cone - cut_min of the plan
    int32_t cut_range;          // phases of the cone
    float mid;                  // centre of the cut values, relative to table value 0
};

struct MemWh {
    int32_t orbit;
    int32_t u, v;               // the term's qubits in the representative's order
    int32_t pad_;
    double W;                   // orbit weight in the group's unit
};

struct WhArgs {
    const GroupWh* groups;      // of one cone size
    const MemWh* mem;
    const uint8_t* cut;
    const double* obs;
    const double* gamma;        // [inst][gamma_P][p]
    const double* beta;
    int64_t gamma_P;
    const double* deltas;
    int32_t p, cut_min;
    int32_t rowcap;             // phases per row in LDS (largest cut_range of the class)
    int32_t realw;
    int32_t P, M;
    int64_t item0, n_items;     // item = group * P + point
    double* zz;                 // [P][M]
    double* g;                  // [P][2p][M]: the group's -2 dE in column rep, zeros in the other members'
};

hipError_t launch_whole(int K, bool grad, const WhArgs& a, hipStream_t st);
// whether the phase rows of a depth-p circuit fit the kernel's LDS
bool whole_fits(int K, int p, int rowcap, bool realw);
// V(x) - sum W / 2 with V(x) = sum over the members of W [x_u != x_v], x with qubit K - 1 = 0, in the
// group's unit (weights of any size then stay in range where the product with psi is rounded to FP32)
hipError_t launch_whole_obs(const GroupWh* groups, int64_t n_groups, const MemWh* mem, int K, double* obs, hipStream_t st);

}  // namespace qaoa
