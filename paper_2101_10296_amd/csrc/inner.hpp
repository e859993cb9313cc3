// Light cones evaluated on their inner qubits: descriptors and launchers (inner.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "depth2.hpp"
#include "shell.hpp"

namespace qaoa {

constexpr int IN_KMIN = 3;     // inner qubits of a cone with a shell at p >= 2
constexpr int IN_KMAX = 10;    // 2^10 amplitudes: 16 per lane of one wave
constexpr int IN_PMAX = 9;     // every layer adds a qubit: p - 1 <= inner - 2
constexpr int IN_ROUNDS = 8;   // rounds of configurations per unit of work

// One light cone: the inner qubits 0 .. kin-1 (closer than p to the edge) carry the state, the
// shell (at distance p) is a sum over configurations.
struct ConeIn {
    int32_t orbit;             // term index m (output column)
    int32_t inst;              // instance of the cone
    int32_t n_grp, grp_off;    // shell groups
    uint32_t nc;               // states of the groups: product of (m_g + 1)
    int32_t tab_off;           // first table in units of 16 bytes
    int32_t kin;               // inner qubits
    int32_t edge_off, n_edges; // cone edges (pairs of qubits, the first the smaller)
    int32_t cfg_off;           // listed configurations, or -1: decoded where they are used
    uint32_t n_cfg;            // listed entries: a whole number of rounds (weight 0 beyond the last)
    uint32_t zmask;            // inner qubits with leaves
    int32_t z_off;             // their leaves: 16 entries from here (zmask 0: none stand there)
    int32_t pad0_;
    double shell_norm;         // 2^-(qubits of the groups)
    int16_t base[IN_PMAX + 1]; // [l], l = 2..p: phase row index of table value 0 of layer l; [1] = [2]
    float mid[IN_PMAX + 1];    // [l]: centre of layer l's cut values, relative to row index 0
    uint8_t mixed[IN_PMAX + 3];// [l]: qubits that layer l mixes (a prefix): those closer than p - l + 1
};

// Shell qubits with the same couplings: only how many of them are 1 matters.
struct GrpIn {
    int32_t m;        // qubits in the group
    int32_t wsum;     // sum of their couplings (one qubit's)
    int32_t h[8];     // coupling to inner qubit 2 + i
};

// One listed configuration: the shifts that the shell makes (see GrpIn) and its weight.
struct alignas(16) CfgList {
    int16_t h[8];
    int32_t c0;
    uint32_t z;                // signs of the qubits with leaves
    double w;
};

struct InArgs {
    const ConeIn* cones;       // cones of this class (inner qubits), from the launch's first
    const CfgList* cfg;
    const GrpIn* grp;
    const ZLeaf* leaf;
    const uint8_t* tab;
    const double* gamma;       // [inst][gamma_P][p]
    const double* beta;
    int64_t gamma_P;
    const double* deltas;
    int32_t signs;             // the class's cones have leaves
    int32_t wz;                // largest coupling of a leaf
    int32_t p, R, cut_min;     // depth; phase row length and the cut value of entry 0
    int32_t P;                 // points of the launch
    int32_t point0;            // first of them
    int32_t M;
    int32_t units;             // units of work per point: cones x chunks
    int32_t chunks;            // units per cone
    int32_t upw;               // units per wave
    int32_t blocks;            // workgroups per point
    // segments of one instance each (the workgroups of one share its phase rows); n_seg > 1:
    // seg[0..n_seg] first unit, then n_seg + 1 first workgroups for this upw, then n_seg instances
    const int32_t* seg;
    int32_t n_seg;
    int32_t inst0;             // n_seg = 1: its instance
    double* zz;                // [P][M], rows from point 0 of the call
    double* g;                 // [P][2p][M]
    double* part;              // chunks > 1: [P of the launch][units][values]
};

// A value of a cone's parts, nv apart, in order.
__device__ __forceinline__ double in_part_sum(const double* src, int chunks, int nv) {
    double x = 0.0;
    int ch = 0;
    for (; ch + 8 <= chunks; ch += 8) {   // eight loads in flight, added in order
        double y[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) y[i] = src[static_cast<size_t>(ch + i) * nv];
#pragma unroll
        for (int i = 0; i < 8; ++i) x += y[i];
    }
    for (; ch < chunks; ++ch) x += src[static_cast<size_t>(ch) * nv];
    return x;
}

hipError_t launch_inner(int kin, bool grad, const InArgs& a, hipStream_t st);
// Small plans (inner_point.hip): the units of a point, a wave each, and where their sums go.
constexpr int IN_POINT = 16;    // units, parts of cones, and orbits, at most
// waves per workgroup: registers for 4 a SIMD; 2 where a wave holds psi and lambda over more
// layers, with its sums in LDS (at most 8 x 19 x 512 bytes)
constexpr int in_point_waves(bool grad, int pp) { return grad && pp == 0 ? 8 : 16; }
constexpr size_t IN_POINT_LDS = 60 << 10;        // phase rows and sums of the gradient at most
// A point of more than four units takes several compute units instead (InPointSum, in two launches) while
// all of a call's units leave half of the chip's 4096 wave slots free: C_1000(1,2,3) at p = 2, 14
// units, energy and gradient at 1, 16, 64, 256 points 42.4, 43.4, 44.9, 51.4 us on a workgroup per
// point, 24.2, 25.3, 28.0, 52.3 spread.
constexpr int64_t IN_SPREAD = 1 << 11;
struct InPoint {
    struct Unit {              // in class order, a cone's parts together
        uint16_t cone, chunk, chunks, part;
        uint8_t kin;
        uint8_t trees;         // 0, or cones in the closed form (depth2_impl.hpp) from `cone` on, a lane each
    } unit[IN_POINT];
    struct Part {              // their values: the parts of a cone together
        uint16_t chunks, orbit;
    } part[IN_POINT];
    int32_t n, n_part;
    const double* W;
    double* energy;
    double* dgamma;
    double* dbeta;
};
// cones of one instance, all with listed configurations; a: cones of the plan, zz and g or null
hipError_t launch_inner_point(const InArgs& a, const D2Args& d, const InPoint& q, bool grad, int64_t n_points, hipStream_t st);

// Workgroups (four units of a class) of a call's small cones, 10 qubits at most, from which these run
// whole, near the crossings for graphs of 9 to 16 nodes.  us per call, inner and whole: 12 nodes with 15
// orbits, p = 2 (6 workgroups a point; with the gradient 5) 1024 points 32 and 44, 64 and 61; 2048
// points 56 and 47, 117 and 71; a path of 13 nodes, p = 3 (4) 1024 points 31 and 37, 95 and 59; 2048
// points 58 and 38, 187 and 64; p = 5 (3) 1024 points 76 and 94, 251 and 210; 4096 points 292 and 175,
// 992 and 532.
constexpr int64_t in_small(int p, bool grad) { return p == 2 ? (grad ? 13 << 9 : 12 << 10) : (grad ? 4 << 10 : 11 << 9); }
// Several classes in one launch (inner_mix.hip), one unit per wave
constexpr int IN_CLASSES = 16;
// Units of a class (over a call's points) that may join: measured faster up to there (16 points of a
// random 4-regular n = 60 168 -> 143 us, 256 points of the cones with cycles of n = 92, 3-regular, 56 ->
// 49, 1024 points 158 -> 145, 4096 points 541 -> 532); beyond, set-up shared by several units per
// wave counts for more.
constexpr int64_t IN_MIX = 1 << 17;
struct InMix {
    struct Class {
        int32_t kin, signs;
        int32_t cone0, n_cones;    // from InArgs::cones on
        int32_t units, chunks;
        int32_t block0;            // first workgroup of a point
        int32_t n_seg, inst0;
        const int32_t* seg;
        int64_t part0;             // its place in the partial sums
        int64_t item0;             // first (point, cone, value) of those that launch_inner_mix_sum adds
    } c[IN_CLASSES];
    int32_t n, blocks;             // workgroups per point
    int32_t all;                   // cones in one unit write partial sums too
    int64_t items;
};
hipError_t launch_inner_mix(const InArgs& a, const InMix& m, bool grad, hipStream_t st);
hipError_t launch_inner_mix_sum(const InArgs& a, const InMix& m, bool grad, hipStream_t st);
// Plans of few cones with many units: the sums of the parts of k_inner_mix and the weighted sums of the
// terms in one launch (inner_point.hip)
struct InPointSum {
    struct Cone {
        int64_t part0;             // its class's place in the partial sums
        int32_t units, unit0;      // of the class per point; the cone's first
        int32_t chunks, orbit;
    } c[IN_POINT];
    int32_t n;
    const double* W;
    double* energy;
    double* dgamma;
    double* dbeta;
};
// a: zz and g or null; n = a.M cones of one instance
hipError_t launch_inner_point_sum(const InArgs& a, const InPointSum& q, bool grad, hipStream_t st);
// sums the chunks of every (point, cone) into zz and g
hipError_t launch_inner_sum(const InArgs& a, int32_t n_cones, bool grad, hipStream_t st);
// Tables of a new plan: of whole cones (cut: a byte per basis state) and of cones on their inner qubits
// (tab: a byte per inner basis state and layer 2 .. p).
struct ConeDev;
struct PlanTabs {
    const ConeDev* cones;
    const ConeIn* in;
    const int32_t* ea;
    const int32_t* eb;
    const int32_t* ew;
    uint8_t* cut;
    uint8_t* tab;
    int64_t n_cones, n_in;
    int32_t p;
    int32_t cut_min;               // of the plan
    uint32_t cut_parts, in_parts;  // set by the launcher
};
hipError_t launch_plan_tables(PlanTabs a, int32_t max_k, hipStream_t st);   // max_k: qubits of the largest of cones

}  // namespace qaoa
