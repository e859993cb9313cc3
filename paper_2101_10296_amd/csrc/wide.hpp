// Light cones on 11 to 14 inner qubits: descriptors and launchers (wide.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "shell.hpp"

namespace qaoa {

constexpr int WD_KMIN = 11;     // inner qubits
constexpr int WD_KMAX = 14;
constexpr int WD_PMAX = 3;
constexpr int WD_CONE2 = 26;    // cone qubits from which this form is used (wide_cone): p = 2
constexpr int WD_CONE3 = 25;    // p = 3
constexpr int WD_NEXT = 8;      // inner qubits that layers 2 and up mix at most
constexpr int WD_CFG = 8;       // configurations per unit of work
constexpr int WD_ROWS = 256;    // phases per row: a cone's cut values span at most 255 units

struct ConeWd {
    int32_t orbit, inst;
    int32_t n_grp, grp_off;     // shell groups (no list)
    uint32_t nc;                // states of the groups
    uint32_t zmask;             // inner qubits with leaves
    int32_t z_off;              // their leaves
    int32_t cfg_off;            // listed configurations, or -1
    uint32_t n_cfg;             // their number (unlisted: half of nc for every choice of signs)
    int32_t first_unit, n_units;
    int32_t edge_off, n_edges;
    int32_t kin;
    int32_t cut_min, n_rows;    // of the cone: cut value of row index 0, phases per row
    int64_t tab_off;            // bytes: tables of layers 2 .. p, 2^kin each
    double shell_norm;
    int16_t base[4];
    float mid[4];
    uint8_t mixed[4];
    uint8_t pad_[4];
};

struct GrpWd {
    int32_t m, wsum;
    int32_t h[12];
};

struct CfgWd {
    int16_t h[12];
    int32_t c0;
    uint32_t z;                 // signs of the qubits with leaves
    double w;
    double dw;                  // (in the kernel) derivative of the weight
};

// One unit: configurations c0 .. c1 - 1 of a cone.
struct UnitWd {
    int32_t cone;
    uint32_t c0, c1;
};

struct WdArgs {
    const ConeWd* cones;        // all of the plan
    const UnitWd* units;        // of this class, from the launch's first
    const GrpWd* grp;
    const CfgWd* cfg;
    const ZLeaf* leaf;
    int32_t wz;                 // largest coupling of a leaf
    const uint8_t* tab;
    const double* gamma;        // [inst][gamma_P][p]
    const double* beta;
    int64_t gamma_P;
    const double* deltas;
    int32_t p;
    int32_t R;                  // phases per row in LDS: the largest n_rows of the plan's cones
    int32_t P, point0;          // points of the launch
    int32_t M;
    int32_t n_units;            // of the launch
    int32_t unit0;              // its first unit's place in the partial sums
    int32_t all_units;          // units of a point's row of partial sums
    int32_t cone0, sum_unit0;   // first cone of that row, and its first unit
    double* part;               // [P][all_units][values]
    double* zz;                 // [..][M], rows from point 0 of the call
    double* g;
};

hipError_t launch_wide(int kin, bool grad, const WdArgs& a, hipStream_t st);
// sums the units of the n_cones cones from cone0 on into zz and g
hipError_t launch_wide_sum(const WdArgs& a, int32_t n_cones, bool grad, hipStream_t st);
hipError_t launch_wide_tables(const ConeWd* cones, int64_t n_cones, const int32_t* ea, const int32_t* eb,
                              const int32_t* ew, int32_t p, uint8_t* tab, hipStream_t st);

}  // namespace qaoa
