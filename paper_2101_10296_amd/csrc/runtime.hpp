// Per-plan device state and the energy driver behind the C ABI.
#pragma once

#include <hip/hip_runtime.h>

#include <string>
#include <vector>

#include "depth1.hpp"
#include "device.hpp"
#include "hbm_impl.hpp"
#include "inner.hpp"
#include "inner_plan.hpp"
#include "plan.hpp"
#include "qaoa.h"
#include "whole.hpp"
#include "wide.hpp"

struct qaoa_plan_s {
    qaoa::HostPlan hp;
    qaoa::PlanOptions opt;

    // ---- device-resident plan data (built on the first energy call, one allocation: d_arena)
    void* d_arena = nullptr;
    int device = -1;
    bool dev_ready = false;
    int32_t max_k = 0;                  // largest cone (qubits)
    struct Group {
        int K;          // cone qubits
        int64_t first;  // first slot in d_cones
        int64_t count;  // cones in this group
        int32_t rowcap; // largest cut range of the group's cones
        // in this order: members of wh_groups that have an inner form only (here for their group's cut
        // table), members with an inner form and this one (in_band), members with this one alone, others
        // in both forms, others in this one
        int64_t n_part[5] = {0, 0, 0, 0, 0};
        int64_t n_in = 0;   // tune = 1 (no wh_groups): the first n_in cones are also in in_groups
    };
    std::vector<Group> lds_groups;      // workgroup-resident cones, grouped by K
    qaoa::ConeDev* d_cones = nullptr;
    uint8_t* d_cut = nullptr;
    // depth-1 plans: every cone, whatever its size, in closed form (in orbit order; sorted by k
    // where a launch covers one cone size or one item: profile, one_cone_at_a_time)
    qaoa::ConeD1* d_d1 = nullptr;
    double2* d_d1w = nullptr;
    std::vector<Group> d1_groups;       // by k (sorted plans), else one group with K = 0
    // cones with a shell and at most IN_KMAX inner qubits, grouped by inner qubits (and by k where
    // launches are timed per cone size: profile, tune = 1)
    struct InGroup {
        int kin, K;         // inner qubits; cone qubits, or 0
        int wh;             // cones that are members of wh_groups: wh_class of their size; else 0
        bool signs;         // cones with leaves (shell.hpp)
        bool tree;          // closed form (depth2.hip): from d_tr + first on, one unit per cone
        int64_t first, count;
        int32_t chunks;     // units of work per cone
        int32_t rounds;     // of configurations of a unit at most (cones outside band 3)
        int32_t small[2];   // workgroups per point that its cones of band 1, of bands 1 and 2 would take alone
        int32_t n_seg;      // instances
        int64_t seg[4];     // n_seg > 1: offset of the segment tables for 1, 2, 4, 8 units per wave
        int32_t blocks[4];  // workgroups per point
    };
    std::vector<InGroup> in_groups;
    // the same classes without the cones of band 1, of bands 1 and 2, of the first one to four sizes of
    // band 3 in in_serial (Forms); classes that hold none of them as above, the others with copies of
    // their descriptors behind the originals
    std::vector<InGroup> in_rest[6];
    std::vector<int> in_serial;         // sizes in band 3, those of most rounds first
    struct Band {           // cones of one size in bands
        int band, wh, K;    // wh: as InGroup
        int64_t count;
        int32_t rounds;     // of one cone at most
    };
    std::vector<Band> in_bands;
    int64_t n_in_cones = 0;             // descriptors in d_in without the copies
    std::vector<int32_t> in_inst;       // instance of each cone in d_in
    qaoa::InPointSum in_parts{};        // few cones in more units than that (n > 0): their parts' places
    qaoa::InPoint in_point{};           // its units where the plan is small enough (n > 0)
    int32_t in_max_k = 0;               // largest of them and of the wide ones (cone qubits)
    // large cones with 11 to 14 inner qubits: units of work by inner qubits (and k: profile)
    struct WdGroup {
        int kin, K;
        int64_t first, count;   // units
    };
    std::vector<WdGroup> wd_groups;
    std::vector<std::pair<int32_t, int32_t>> wd_units;   // (first unit, units) of each cone
    int64_t wd_all_units = 0, wd_most_units = 0;   // of the plan, of one cone
    int32_t wd_rows = 1;                // phases per row of the largest cut range
    qaoa::ConeWd* d_wd = nullptr;
    qaoa::UnitWd* d_wdunit = nullptr;
    qaoa::GrpWd* d_wdgrp = nullptr;
    qaoa::ZLeaf* d_wdleaf = nullptr;
    qaoa::ZLeaf* d_leaf = nullptr;       // of the cones in d_in
    int32_t wz = 0;                      // largest coupling of a leaf
    qaoa::D2Cone* d_tr = nullptr;        // depth-2 trees
    qaoa::D2SideDef* d_sides = nullptr;
    int32_t n_sides = 0;
    int32_t* d_branch = nullptr;
    qaoa::D2Type* d_types = nullptr;
    qaoa::D2Leaf* d_leaf2 = nullptr;
    std::vector<int32_t> tr_inst;        // instance of each
    bool d2_point = false;               // all cones are trees, few enough for one launch per call
    int32_t n_types = 0;
    qaoa::CfgWd* d_wdcfg = nullptr;
    uint8_t* d_wdtab = nullptr;
    qaoa::ConeIn* d_in = nullptr;
    qaoa::GrpIn* d_ingrp = nullptr;
    qaoa::CfgList* d_incfg = nullptr;
    uint8_t* d_intab = nullptr;
    int32_t* d_inseg = nullptr;
    size_t cap_part = 0;
    double* d_part = nullptr;           // partial sums of cones in several units
    // groups of cones with the same qubits, by k: they share one state wherever the caller does not
    // ask for every term's own gradient (such calls take the members' own forms)
    struct WhGroup {
        int K;
        int64_t first, count;   // groups
        int64_t members;        // their cones
        int32_t rowcap;
    };
    std::vector<WhGroup> wh_groups;
    qaoa::GroupWh* d_wh = nullptr;
    qaoa::MemWh* d_whmem = nullptr;
    double* d_whobs = nullptr;
    // orbit weights of the gradient sums, for every choice of classes that share their states (bit 0: 13
    // qubits, bit 1: 14; up to 12 always): 1 at a sharing group's column, 0 at its other members
    double* d_Wg = nullptr;
    // HBM-resident cones, grouped by k
    struct HGroup {
        int K;
        int64_t first;
        int64_t count;
        int32_t rowcap;
    };
    std::vector<HGroup> hbm_groups;
    qaoa::ConeHbm* d_hcones = nullptr;
    int32_t *d_ea = nullptr, *d_eb = nullptr, *d_ew = nullptr;
    double* d_ewd = nullptr;            // real weights of the cone edges (real-weight plans)
    uint8_t* d_tt = nullptr;
    double* d_W = nullptr;
    int64_t* d_inst_orbit = nullptr;    // [n_inst + 1]
    double* d_inst_delta = nullptr;     // [n_inst]
    double* d_ones = nullptr;           // [n_inst] of 1.0 (combination of per-term gradients in radians)
    size_t resident_bytes = 0;

    // ---- profiling (opts.profile): events around each kernel group of the last call
    struct Timed {
        int32_t k;
        int64_t items;
        hipEvent_t start, stop;
    };
    std::vector<Timed> timed;
    size_t n_timed = 0;

    // ---- per-call scratch, grown on demand
    size_t cap_phase = 0, cap_mix = 0, cap_zz = 0, cap_g = 0;
    float2* d_phase = nullptr;
    float2* d_mix = nullptr;
    double* d_zz = nullptr;
    double* d_g = nullptr;
    size_t cap_phi = 0, cap_lam = 0, cap_gpart = 0;
    float2* d_phi = nullptr;
    float2* d_lam = nullptr;
    double* d_gpart = nullptr;
    std::vector<int64_t> hbm_batch;     // items per batch of each HBM group in the last call
    std::vector<int8_t> hbm_ckpt;       // 1 if the HBM group stored forward checkpoints in the last call
    int64_t pass_launches[qaoa::N_PASS_KINDS] = {};   // per pass kind, last eager call
    int32_t checkpointed_classes = 0;   // HBM groups that stored checkpoints in the last eager call
    uint32_t checkpointed_k_mask = 0;   // bit k: the k-qubit class did

    // ---- graph replay (opts.graph)
    struct GraphKey {
        int64_t n_points = -1;
        bool grad = false;
        const void* ptr[7] = {nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr};
        bool operator==(const GraphKey& o) const {
            if (n_points != o.n_points || grad != o.grad) return false;
            for (int i = 0; i < 7; ++i)
                if (ptr[i] != o.ptr[i]) return false;
            return true;
        }
    };
    GraphKey gkey;
    hipGraphExec_t gexec = nullptr;
    int64_t graph_replays = 0;
    hipStream_t cap_stream = nullptr;
};

namespace qaoa {

qaoa_status run_energy(qaoa_plan_s* plan, int64_t n_points, const double* gamma, const double* beta,
                       double* energy, double* term_zz, double* dgamma, double* dbeta, double* term_grad,
                       hipStream_t stream,
                       std::string& msg);

// Depth-1 plans evaluated in closed form; tune = 2..5 asks for a layout of the statevector kernel.
inline bool depth1_closed(const qaoa_plan_s* P) { return P->hp.p == 1 && P->opt.tune < 2; }

// Cones evaluated on their inner qubits: those with a shell (else there is nothing to average
// over, and the kernels for whole cones store half of the state) whose inner state fits the
// registers of one wave.  Measured against those kernels: 14 qubits, p = 2 (6 inner) 93x, 18 qubits
// (8 inner) 4x, 26 qubits (8 inner) 150x; C_10000(1,2) at one point, 10-11 qubits with as many
// amplitudes as before, 26.7 -> 16 us for the call.  Cones of up to 14 qubits where it depends on the
// call are held in both forms (in_band, choose_forms).  Real weights (but for depth-2 trees) and
// forced layouts (tune >= 2) keep the kernels for whole cones.
inline bool inner_cone(const qaoa_plan_s* P, const Cone& c) {
    const int32_t p = P->hp.p;
    return p >= 2 && p <= IN_PMAX && P->opt.tune < 2 && c.nd[p - 1] <= IN_KMAX && c.nd[p - 1] < c.k &&
           (!P->hp.realw || (p == 2 && tree_cone(c, true)));
}

// Those of them in the closed form of depth2_impl.hpp (a term of a 14-qubit cone: 0.6 ns as states of
// its 6 inner qubits, 0.03 ns).  Up to 10 inner qubits, as for the states: the tests hold the pass
// kinds that larger cones launch.
inline bool closed_tree(const qaoa_plan_s* P, const Cone& c) {
    return P->hp.p == 2 && inner_cone(P, c) && tree_cone(c, P->hp.realw);
}

// Cones with more inner qubits, on a workgroup each.  The lines at 26 (p = 2) and 25 cone qubits
// (p = 3) are not where the passes over device memory get faster.  Measured with the gradient at
// p = 3: a 25-qubit cone costs the passes 763 us against 92, a 24-qubit one 385 against 22, a 20-qubit
// one with 15 inner qubits 56 against 74.  The tests hold the pass kinds of cones of 23 and 25 qubits at
// p = 2 and of 24 at p = 3; nothing but these lines keeps 21 to 23 qubits at p = 3 on the passes.
// Above lies nearly all of the work: a cone's cost doubles per qubit.
inline bool wide_cone(const qaoa_plan_s* P, const Cone& c) {
    const int32_t p = P->hp.p;
    return p >= 2 && p <= WD_PMAX && !P->hp.realw && P->opt.tune < 2 &&
           c.k >= (p == 2 ? WD_CONE2 : WD_CONE3) && c.nd[p - 1] >= WD_KMIN &&
           c.nd[p - 1] <= WD_KMAX && c.nd[p - 2] <= WD_NEXT && c.nd[p - 1] < c.k;
}

// Sizes of shared states with a line of their own.
inline int wh_class(int K) { return K <= 12 ? 12 : K; }

// Which groups of wh_groups a call evaluates on their shared state.
struct Shared {
    bool on[3] = {};         // wh_class 12, 13, 14
    const double* Wg;        // weights of the gradient sums
    bool of(int cls) const { return cls != 0 && on[cls - 12]; }   // cls: wh_class, or 0
};
Shared shared_states(const qaoa_plan_s* P, bool grad, bool terms_read, int64_t n_points);

// Cones of up to k_lds_max qubits with an inner form that is not always the faster one (no trees, which
// are in closed form): 1 up to 9 qubits, 2 of 10, 3 of 11 to 14 that take several rounds of
// configurations; 0: always the inner form.  A call chooses one form for each band (whole_forms).
inline int in_band(const qaoa_plan_s* P, const Cone& c, bool tree, uint32_t rounds) {
    if (P->opt.tune != 0 || tree || c.k > P->opt.k_lds_max) return 0;
    return c.k <= 9 ? 1 : c.k == 10 ? 2 : rounds >= 2 ? 3 : 0;
}

// What a call runs in which form.
struct Forms {
    Shared sh;
    uint32_t whole = 0;      // sizes whose cones in bands run on the kernel for whole cones: a bit each
    const std::vector<qaoa_plan_s::InGroup>* in = nullptr;   // classes on their inner qubits, but for those that share
    // runs [begin, end) of a size's cones on the kernel for whole cones: at most two
    int runs(const qaoa_plan_s::Group& g, int64_t (&r)[2][2]) const;
};
Forms choose_forms(const qaoa_plan_s* P, bool grad, bool terms_read, int64_t n_points);
hipError_t launch_whole_group(const qaoa_plan_s* P, const qaoa_plan_s::WhGroup& grp, bool grad, int64_t n_points,
                              const double* gamma, const double* beta, int64_t gamma_P, double* zz, double* g,
                              hipStream_t st);

// One class of them (grp) for a call's points: terms into zz, g; part: room for the partial sums of
// at least one point (null where every cone is one unit).
hipError_t launch_inner_group(const qaoa_plan_s* P, const qaoa_plan_s::InGroup& grp, bool grad, int upw_log2,
                              int64_t n_points, const double* gamma, const double* beta, int64_t gamma_P, double* zz,
                              double* g, double* part, size_t part_cap, hipStream_t st);

void release_device(qaoa_plan_s* plan);

// The run-time tuner's choices so far (one line per kernel class).
std::string tuning_report();

// Records msg as this thread's last error (capi.hip) and returns st.
qaoa_status set_last_error(qaoa_status st, const std::string& msg);
void clear_last_error();
qaoa_status kernel_times(qaoa_plan_s* plan, int32_t cap, int32_t* k_out, int64_t* items_out, double* ms_out,
                         int32_t* n_out, std::string& msg);

// kernel launchers
// variant: layout of the workgroup kernel (0 default; see Fz in fused_impl.hpp)
hipError_t launch_fused(int K, bool grad, int variant, const ConeDev* cones, int64_t item_base, int64_t n_items,
                        const uint8_t* cut, int32_t rowcap, const EvalArgs& ea, hipStream_t st);
std::vector<int> fused_variants(int K, bool grad);
hipError_t launch_tables(const double* gamma, const double* beta, int64_t n_pl, int32_t R, int32_t cmin,
                         const double* deltas, int64_t pl_per_inst, float2* phase, float2* mix, hipStream_t st);
hipError_t launch_cut_tables_real(const ConeDev* cones, int64_t n_cones, const int32_t* ea, const int32_t* eb,
                                  const double* ew, float* tables, hipStream_t st);
hipError_t launch_pass(int kind, const PassArgs& pa, hipStream_t st);
hipError_t launch_tt_tables(const ConeHbm* cones, int64_t n_cones, int max_groups, const int32_t* ea,
                            const int32_t* eb, const int32_t* ew, uint8_t* tt, hipStream_t st);
hipError_t launch_tt_tables_real(const ConeHbm* cones, int64_t n_cones, int max_groups, const int32_t* ea,
                                 const int32_t* eb, const double* ew, float* tt, hipStream_t st);
hipError_t launch_fill_zero(double* x, int64_t n, hipStream_t st);
hipError_t launch_tile_reduce(const ConeHbm* cones, const double* gpart, int64_t item0, int64_t n_batch,
                              int64_t tiles, int32_t stride, int32_t nvals, const EvalArgs& ea, hipStream_t st);

// One pass of the HBM program (see hbm_impl.hpp).
struct PassSpec {
    int kind, group, la, lb, m0a, m0b;
    int fix_layer = 0, fix_pow = 0;   // rescaling of psi read as the forward sweep left it
    int ck_in = -1, ck_out = -1;      // checkpoint slots read / written (-1: the single state buffer)
    int store_phi = 1;                // reverse passes: write the undone psi back
};
int hbm_groups_of(int k);
int hbm_group_qubits(int k, int grp);
// ckpt: every forward pass but the final one writes its output to a slot of its own
// (hbm_checkpoints(k, p) slots) and every reverse pass reads psi from the slot of the
// forward pass it undoes instead of carrying the uncomputed psi along.
std::vector<PassSpec> hbm_program(int k, int p, bool grad, bool ckpt = false);
int hbm_checkpoints(int k, int p);

hipError_t launch_scale_gamma_terms(double* g, int64_t P, int32_t p, int32_t M, const int64_t* inst_orbit,
                                    int32_t n_inst, const double* deltas, hipStream_t st);
// points per k_combine launch with ny blocks per point (grid below 2^32 work-items)
int64_t combine_chunk(uint32_t ny);
// energy [n_inst][P_out], dgamma / dbeta [n_inst][P_out][p]: points i0 .. i0 + Pc - 1 of
// each instance from the term rows zz [Pc][M] (weights W) and g [Pc][2p][M] (weights Wg)
hipError_t launch_combine(const double* W, const double* Wg, const double* zz, const double* g, int32_t M, int32_t p,
                          const int64_t* inst_orbit, const double* deltas, int32_t n_inst, int64_t Pc,
                          int64_t P_out, int64_t i0, double* energy, double* dgamma, double* dbeta, hipStream_t st);

}  // namespace qaoa
