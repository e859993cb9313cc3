// Host planning of cones evaluated on their inner qubits: the order of the inner qubits, their layer
// prefixes, the shell's groups and the configurations of the shell up to symmetry.
#pragma once

#include <cstdint>
#include <vector>

#include "plan.hpp"
#include "shell_limits.hpp"

namespace qaoa {

constexpr int SH_KMAX = 14;    // inner qubits
constexpr int SH_H = 12;       // of them next to the shell (never u or v): qubits 2 .. 13

// Shell qubits with the same couplings: only how many of them are 1 matters.
struct ShellGroup {
    int32_t m = 0;             // qubits
    int32_t wsum = 0;          // sum of one qubit's couplings
    int32_t h[SH_H] = {};      // coupling to inner qubit 2 + i
};

// The shell qubits that couple to one inner qubit only, two or more of them: m[i] of coupling
// +-w[i] (see shell.hpp; a qubit with more than ZL_W different couplings keeps them as groups).
struct ShellLeaves {
    int16_t w[ZL_W] = {};
    int16_t m[ZL_W] = {};
};

// One configuration up to symmetry: c0 + sum_a x_a h_a is what the shell's groups add to C_in(x), and
// z the signs of the inner qubits with leaves.
struct ShellCfg {
    int16_t h[SH_H] = {};
    int32_t c0 = 0;
    uint32_t z = 0;
    double w = 0.0;            // configurations that it stands for
};

// A cone's inner qubits in an order of their own (by distance, then next to the qubits before them),
// so that cones of one shape agree in their couplings.
struct ShellCone {
    int32_t kin = 0;
    int64_t edge = 0;          // couplings with an inner end, in that order (ea < eb): ShellPlanner's arrays
    int32_t n_edges = 0;
    uint32_t nc = 0;           // states of the groups: product of (m + 1), at most 2^28
    uint32_t zmask = 0;        // inner qubits with leaves
    // a tree (see ShellPlanner): the edge's coupling and the neighbours of u, then of v, from `br` on
    bool tree = false;
    int16_t nu = 0, nv = 0;
    int32_t br = 0;
    double w_uv = 0.0;
    int32_t n_leaf = 0;        // their leaves
    int32_t w_leaf = 0;        // and the sum of the couplings
    uint32_t runs() const { return ((nc + 1) / 2) << __builtin_popcount(zmask); }   // without a list
    int32_t shape = -1;        // cones of one shape share groups and configurations
};

// A neighbour of u or v and its leaves.  Integer couplings of the neighbour up to +-3 and of at most six
// leaves up to +-3 have a code: (w + 3) 343 + n_1 + 7 n_2 + 49 n_3, n_x leaves of coupling +-x.
constexpr int SH_CODES = 7 * 343;
struct ShellBranch {
    double w = 0.0;
    int16_t code = -1;
    int16_t n_leaf = 0;        // code < 0: couplings leaf_w[leaf ..]
    int32_t leaf = 0;
};

class ShellPlanner {
public:
    // trees: cones whose inner qubits couple to u or v alone and whose shell qubits are leaves get no
    // shape but a list of branches; real: couplings are Cone::wf (then every cone has to be a tree)
    explicit ShellPlanner(int32_t p, bool trees = false, bool real = false) : p_(p), trees_(trees), real_(real) {}
    // the cones in order (0.6 us of host time each: on several threads from 4096 cones on)
    void add(const std::vector<const Cone*>& cones, std::vector<ShellCone>& out);
    // Lists the configurations of every shape seen so far that has none yet (several threads).
    void list();
    // null: no list, every configuration is run
    const std::vector<ShellCfg>* configurations(int32_t shape) const;
    const ShellLeaves* leaves(int32_t shape) const { return shapes_[static_cast<size_t>(shape)].leaf; }   // [SH_KMAX]
    const std::vector<ShellGroup>& groups(int32_t shape) const { return shapes_[static_cast<size_t>(shape)].grp; }
    std::vector<int32_t> ea, eb, ew;   // couplings of all cones
    std::vector<ShellBranch> branches; // of all trees
    std::vector<double> leaf_w;        // the couplings of leaves without a code

private:
    struct Shape {
        int kin = 0;
        uint8_t level[SH_KMAX] = {};      // distance of each inner qubit
        int16_t w[SH_KMAX][SH_KMAX] = {}; // couplings between inner qubits
        std::vector<ShellGroup> grp;
        ShellLeaves leaf[SH_KMAX];
        uint32_t zmask = 0;
        uint32_t nc = 0;
        uint64_t hash = 0;
        bool listed = false;
        std::vector<ShellCfg> cfg;
        bool same(const Shape& o) const;
        void enumerate();
    };
    int32_t p_;
    bool trees_, real_;
    std::vector<Shape> shapes_;
    std::vector<std::pair<uint64_t, int32_t>> table_;   // open addressing by hash
    Shape s_;                                            // the cone being added
    int32_t find(uint64_t h);                            // shape of s_
    void add_one(const Cone& c, ShellCone& out);
    bool add_tree(const Cone& c, ShellCone& out);
};

// Whether a depth-2 cone with a shell is a tree in that sense.
bool tree_cone(const Cone& c, bool real);

}  // namespace qaoa
