// Device runtime of a plan: one-time upload of cone descriptors and cut tables, scratch
// management, and the sequence of launches of one energy (and gradient) evaluation.
#include "runtime.hpp"

#include "inner_plan.hpp"

#include <algorithm>
#include <array>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <map>
#include <mutex>
#include <numeric>
#include <tuple>

namespace qaoa {
namespace {

// ---- run-time tuner (plans built with opts.tune = 1).  Layout choices of a kernel class
// are timed once per process on the first call that needs them (HIP events on the call's
// stream) and the fastest is kept, keyed by (device architecture, what, k, p, gradient,
// real weights, form).  form: which of the size's cones run on their inner qubits, and how many
// those are (empty: none): their time says nothing about cones in another form.  what = 0: register bits per LDS stage / workgroup size of the
// workgroup-resident kernel (fused_variants); what = 1: tiles per workgroup of the
// device-memory passes; what = 2: units per wave of cones above k_lds_max qubits that run on
// their inner qubits (reported under the name of 1: such a unit stands where a tile stood).
struct TuneKey {
    std::string arch;
    int what, k, p, grad, realw;
    std::string form;
    bool operator<(const TuneKey& o) const {
        return std::tie(arch, what, k, p, grad, realw, form) <
               std::tie(o.arch, o.what, o.k, o.p, o.grad, o.realw, o.form);
    }
};
struct TuneRec {
    int choice = 0;
    std::vector<std::pair<int, float>> ms;   // candidate -> milliseconds per timed launch
    int64_t items = 0;                       // items of the timed launches
};
std::mutex g_tune_mu;
std::map<TuneKey, TuneRec> g_tune;

std::string device_arch(int dev) {
    static std::mutex mu;
    static std::map<int, std::string> names;
    std::lock_guard<std::mutex> lk(mu);
    auto it = names.find(dev);
    if (it != names.end()) return it->second;
    hipDeviceProp_t prop{};
    std::string a = hipGetDeviceProperties(&prop, dev) == hipSuccess ? std::string(prop.gcnArchName) : "unknown";
    names[dev] = a;
    return a;
}

bool tune_lookup(const TuneKey& key, int& choice) {
    std::lock_guard<std::mutex> lk(g_tune_mu);
    auto it = g_tune.find(key);
    if (it == g_tune.end()) return false;
    choice = it->second.choice;
    return true;
}

// Times run(candidate) for every candidate (one untimed launch, then `reps` timed ones on
// the stream) and records the fastest under key.
template <class Run>
hipError_t tune_pick(const TuneKey& key, const std::vector<int>& cand, int64_t items, hipStream_t st, Run&& run,
                     int& choice) {
    TuneRec rec;
    rec.items = items;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    hipError_t e = hipEventCreate(&e0);
    if (e == hipSuccess) e = hipEventCreate(&e1);
    constexpr int reps = 3;
    float best = 0.f;
    for (size_t i = 0; e == hipSuccess && i < cand.size(); ++i) {
        e = run(cand[i]);
        if (e == hipSuccess) e = hipEventRecord(e0, st);
        for (int r = 0; e == hipSuccess && r < reps; ++r) e = run(cand[i]);
        if (e == hipSuccess) e = hipEventRecord(e1, st);
        if (e == hipSuccess) e = hipEventSynchronize(e1);
        float ms = 0.f;
        if (e == hipSuccess) e = hipEventElapsedTime(&ms, e0, e1);
        if (e != hipSuccess) break;
        ms /= reps;
        rec.ms.emplace_back(cand[i], ms);
        if (i == 0 || ms < best) {
            best = ms;
            rec.choice = cand[i];
        }
    }
    if (e0) hipEventDestroy(e0);
    if (e1) hipEventDestroy(e1);
    if (e != hipSuccess) return e;
    choice = rec.choice;
    std::lock_guard<std::mutex> lk(g_tune_mu);
    g_tune[key] = rec;
    return hipSuccess;
}

#define QCHECK(expr)                                                               \
    do {                                                                           \
        hipError_t e_ = (expr);                                                    \
        if (e_ != hipSuccess) {                                                    \
            msg = std::string(#expr) + ": " + hipGetErrorString(e_);               \
            return (e_ == hipErrorOutOfMemory) ? QAOA_ENOMEM : QAOA_EHIP;         \
        }                                                                          \
    } while (0)

template <class T>
qaoa_status grow(T*& ptr, size_t& cap, size_t need, std::string& msg) {
    if (need <= cap && ptr) return QAOA_OK;
    if (ptr) {
        hipFree(ptr);
        ptr = nullptr;
        cap = 0;
    }
    const size_t bytes = std::max<size_t>(need, 1) * sizeof(T);
    hipError_t e = hipMalloc(reinterpret_cast<void**>(&ptr), bytes);
    if (e != hipSuccess) {
        (void)hipGetLastError();   // clear the failure so later launch checks do not see it
        ptr = nullptr;
        msg = "device allocation of " + std::to_string(bytes) + " bytes failed: " + hipGetErrorString(e);
        return QAOA_ENOMEM;
    }
    cap = std::max<size_t>(need, 1);
    return QAOA_OK;
}

// Pass groups over the kh = k - 1 stored qubits of a k-qubit HBM cone: group 0 = qubits
// 0..12, group j >= 1 = nine of the remaining qubits; tile bit i of group g maps to global
// bit hbm_group_global_bit(kh, g, i) (the same map as hgroup_bits in hbm_impl.hpp).
int hbm_group_global_bit(int k, int grp, int i) {
    if (grp == 0) return i;
    const int lo = 13 + 9 * (grp - 1);
    const int h = std::min(k, lo + 9) - lo;
    if (i < h) return lo + i;
    if (i < 9) return 4 + (i - h);
    return i - 9;
}

}  // namespace

int hbm_groups_of(int k) { return 1 + (k - 13 + 8) / 9; }

int hbm_group_qubits(int k, int grp) {
    if (grp == 0) return 13;
    const int lo = 13 + 9 * (grp - 1);
    return std::min(k, lo + 9) - lo;
}

int hbm_checkpoints(int k, int p) {
    return p == 1 ? 0 : 1 + (p - 1) * (hbm_groups_of(k - 1) - 1) - 1;
}

// Forward program over the stored qubits (kh = k - 1): layer l (1 <= l <= p-1) visits the
// groups in descending order when p-1-l is even, ascending otherwise, so layer p-1 ends on
// group 0 and consecutive layers share a pass.  Group-0 passes also mix the dropped qubit
// k-1 (14 qubits per layer).  With grad, the last pass is the fused final/adjoint pass and
// the earlier passes follow in reverse as RV_* passes; m0a / m0b count the qubits of a
// layer already undone by earlier reverse passes.
std::vector<PassSpec> hbm_program(int k, int p, bool grad, bool ckpt) {
    std::vector<PassSpec> fwd;
    const int kh = k - 1;
    const int n = hbm_groups_of(kh);
    auto layer_qubits = [&](int g) { return hbm_group_qubits(kh, g) + (g == 0 ? 1 : 0); };
    if (p == 1) {
        fwd.push_back({grad ? GR_GEN_FINAL : FWD_GEN_FINAL, 0, 0, 1, 0, 0});
        return fwd;
    }
    ckpt = ckpt && grad;
    auto group_at = [&](int l, int j) { return (((p - 1 - l) & 1) == 0) ? n - 1 - j : j; };
    // in_prog[i] / mixed[i]: the layer in progress after forward pass i and how many of its
    // qubits have been mixed by then (the forward scale of the state written by pass i)
    std::vector<int> in_prog, mixed;
    fwd.push_back({FWD_GEN_MIX, group_at(1, 0), 0, 1, 0, 0});
    in_prog.push_back(1);
    mixed.push_back(layer_qubits(fwd.back().group));
    for (int l = 1; l <= p - 1; ++l)
        for (int j = 1; j < n; ++j) {
            const int g = group_at(l, j);
            if (j < n - 1) {
                fwd.push_back({FWD_MIX, g, l, 0, 0, 0});
                in_prog.push_back(l);
                mixed.push_back(mixed.back() + layer_qubits(g));
            } else if (l + 1 <= p - 1) {
                fwd.push_back({FWD_BND_MIX, g, l, l + 1, 0, 0});
                in_prog.push_back(l + 1);
                mixed.push_back(layer_qubits(g));
            } else {
                fwd.push_back({FWD_BND_FINAL, g, l, p, 0, 0});
            }
        }
    const int nf = static_cast<int>(fwd.size()) - 1;   // forward passes before the final one
    if (ckpt)
        for (int i = 0; i <= nf; ++i) {
            fwd[i].ck_in = i - 1;
            fwd[i].ck_out = i < nf ? i : -1;
        }
    if (!grad) return fwd;
    std::vector<PassSpec> out(fwd.begin(), fwd.end() - 1);
    std::vector<int> undone(p + 2, 0);
    PassSpec fin = fwd.back();
    fin.kind = GR_BND_FINAL;
    fin.m0a = undone[fin.la];
    undone[fin.la] += layer_qubits(fin.group);
    out.push_back(fin);
    for (int i = nf - 1; i >= 0; --i) {
        PassSpec r = fwd[i];
        const int h = layer_qubits(r.group);
        if (r.kind == FWD_GEN_MIX) {
            r.kind = RV_GEN_MIX;
            r.m0b = undone[r.lb];
            undone[r.lb] += h;
        } else if (r.kind == FWD_MIX) {
            r.kind = RV_MIX;
            r.m0a = undone[r.la];
            undone[r.la] += h;
        } else {
            r.kind = RV_BND_MIX;
            r.m0b = undone[r.lb];
            undone[r.lb] += h;
            r.m0a = undone[r.la];
            undone[r.la] += h;
        }
        if (ckpt || i == nf - 1) {
            // psi read as the forward sweep left it (pass i's output): rescale it from the
            // forward scale of its layer in progress to lambda's
            r.fix_layer = in_prog[i];
            r.fix_pow = 2 * mixed[i] - k;
        }
        if (ckpt) {
            r.ck_in = i;
            r.ck_out = -1;
            r.store_phi = 0;
        }
        out.push_back(r);
    }
    return out;
}

namespace {

// pinned staging buffer of the plan uploads (ensure_device)
std::mutex g_stage_mu;
void* g_stage = nullptr;
size_t g_stage_cap = 0;

// Groups of at least WH_MEMBERS cones with the same qubits (whole.hpp).
struct WholeHost {
    std::vector<char> member;    // per orbit; empty: none
    std::vector<GroupWh> groups;
    std::vector<MemWh> mem;
    std::vector<double> Wg;      // see qaoa_plan_s::d_Wg
    int64_t obs = 0;             // entries of the observable tables
};

void build_whole(qaoa_plan_s* P, WholeHost& w) {
    const HostPlan& hp = P->hp;
    P->wh_groups.clear();
    if (hp.p < 2 || P->opt.tune != 0) return;   // layouts of the cones on their own are asked for
    // cones of one size whose node ids agree in a commutative hash (counted in a table, as nearly
    // all cones of a large graph are alone), then exactly
    struct Key {
        int32_t k;
        uint64_t h;
        int64_t m;
    };
    const size_t n = hp.cones.size();
    size_t cap = 64;
    while (cap < 2 * n) cap *= 2;
    std::vector<uint64_t> hash(n, 0), slot(cap, 0);
    std::vector<int32_t> count(cap, 0);
    auto at = [&](uint64_t h) {
        size_t i = (h >> 20) & (cap - 1);
        while (count[i] && slot[i] != h) i = (i + 1) & (cap - 1);
        return i;
    };
    for (size_t m = 0; m < n; ++m) {
        const Cone& c = hp.cones[m];
        if (c.k < WH_KMIN || c.k > WH_KMAX) continue;
        uint64_t h = static_cast<uint64_t>(c.k);
        for (int32_t x : c.nodes) {
            uint64_t z = static_cast<uint64_t>(x) * 0x9E3779B97F4A7C15ull + 0x632BE59BD9B4E019ull;
            z ^= z >> 29;
            h += z * 0xBF58476D1CE4E5B9ull;
        }
        hash[m] = h;
        const size_t i = at(h);
        slot[i] = h;
        ++count[i];
    }
    std::vector<Key> keys;
    for (size_t m = 0; m < n; ++m)
        if (hash[m] && count[at(hash[m])] >= WH_MEMBERS && !closed_tree(P, hp.cones[m])) keys.push_back({hp.cones[m].k, hash[m], static_cast<int64_t>(m)});
    std::sort(keys.begin(), keys.end(), [](const Key& a, const Key& b) {
        return std::tie(a.k, a.h, a.m) < std::tie(b.k, b.h, b.m);
    });
    auto nodes = [&](int64_t m) {
        std::vector<int32_t> v = hp.cones[static_cast<size_t>(m)].nodes;
        std::sort(v.begin(), v.end());
        return v;
    };
    for (size_t i = 0, j; i < keys.size(); i = j) {
        for (j = i + 1; j < keys.size() && keys[j].k == keys[i].k && keys[j].h == keys[i].h; ++j) {}
        if (j - i < WH_MEMBERS) continue;
        const int64_t rep = keys[i].m;
        const Cone& c = hp.cones[static_cast<size_t>(rep)];
        const std::vector<int32_t> want = nodes(rep);
        GroupWh g{};
        g.inst = c.inst;
        g.rep = static_cast<int32_t>(rep);
        g.mem_off = static_cast<int32_t>(w.mem.size());
        for (size_t q = i; q < j; ++q) {
            if (nodes(keys[q].m) != want) continue;   // a hash collision: stays on its own
            const Cone& x = hp.cones[static_cast<size_t>(keys[q].m)];
            MemWh e{};
            e.orbit = static_cast<int32_t>(keys[q].m);
            e.u = static_cast<int32_t>(std::find(c.nodes.begin(), c.nodes.end(), x.nodes[0]) - c.nodes.begin());
            e.v = static_cast<int32_t>(std::find(c.nodes.begin(), c.nodes.end(), x.nodes[1]) - c.nodes.begin());
            e.W = hp.W[static_cast<size_t>(keys[q].m)];
            w.mem.push_back(e);
        }
        g.n_mem = static_cast<int32_t>(w.mem.size()) - g.mem_off;
        const int32_t range = hp.realw ? 1 : c.cut_max - c.cut_min + 1;
        if (g.n_mem < WH_MEMBERS || !whole_fits(c.k, hp.p, range, hp.realw)) {
            w.mem.resize(static_cast<size_t>(g.mem_off));
            continue;
        }
        g.cut_row = hp.realw ? 0 : c.cut_min - hp.cut_min;
        g.cut_range = range;
        g.mid = static_cast<float>(0.5 * (range - 1));
        double most = 0.0;
        for (size_t q = static_cast<size_t>(g.mem_off); q < w.mem.size(); ++q) most = std::max(most, std::fabs(w.mem[q].W));
        const int unit = most > 0.0 ? std::ilogb(most) : 0;
        g.scale = std::ldexp(1.0, unit);
        for (size_t q = static_cast<size_t>(g.mem_off); q < w.mem.size(); ++q) w.mem[q].W = std::ldexp(w.mem[q].W, -unit);
        g.v_off = w.obs;
        w.obs += int64_t{1} << (c.k - 1);
        if (P->wh_groups.empty() || P->wh_groups.back().K != c.k)
            P->wh_groups.push_back({c.k, static_cast<int64_t>(w.groups.size()), 0, 0, 1});
        auto& cls = P->wh_groups.back();
        cls.count += 1;
        cls.members += g.n_mem;
        cls.rowcap = std::max(cls.rowcap, range);
        w.groups.push_back(g);
    }
    if (w.groups.empty()) return;
    w.member.assign(hp.cones.size(), 0);
    for (const MemWh& e : w.mem) w.member[static_cast<size_t>(e.orbit)] = 1;
    for (int sel = 0; sel < (P->wh_groups.back().K > 12 ? 4 : 1); ++sel) {
        w.Wg.insert(w.Wg.end(), hp.W.begin(), hp.W.end());
        double* Wg = w.Wg.data() + static_cast<size_t>(sel) * hp.W.size();
        for (const auto& cls : P->wh_groups) {
            if (cls.K > 12 && !((sel >> (cls.K - 13)) & 1)) continue;
            for (int64_t i = cls.first; i < cls.first + cls.count; ++i) {
                const GroupWh& g = w.groups[static_cast<size_t>(i)];
                for (int32_t m = g.mem_off; m < g.mem_off + g.n_mem; ++m) Wg[w.mem[static_cast<size_t>(m)].orbit] = 0.0;
                Wg[g.rep] = 1.0;
            }
        }
    }
}

// Descriptors of the cones evaluated on their inner qubits (inner.hpp).
struct InnerHost {
    std::vector<ConeIn> cones;
    std::vector<GrpIn> grp;
    std::vector<int32_t> seg;
    std::vector<CfgList> cfg;
    std::vector<ZLeaf> leaf;
    std::vector<D2Cone> tr;
    std::vector<int32_t> branch;
    std::vector<D2SideDef> sides;
    std::vector<D2Type> types;
    std::vector<D2Leaf> leaf2;
    int64_t tab_units = 0;   // table bytes / 16
    std::vector<char> band;  // in_band of every orbit
};

// Configurations that a wave runs at once, and the rounds of them that a cone takes.
uint32_t shell_at_once(const ShellCone& q) { return 64u >> std::max(0, q.kin - 4); }
uint32_t shell_rounds(const ShellPlanner& sp, const ShellCone& q) {
    const std::vector<ShellCfg>* list = sp.configurations(q.shape);
    return ((list ? static_cast<uint32_t>(list->size()) : q.runs()) + shell_at_once(q) - 1) / shell_at_once(q);
}

// Mixed prefixes and cut ranges of every layer: base = phase row index of the smallest cut value of the
// couplings inside the qubits mixed by layer l - 1, mid = centre of the layer's cut values in
// row indices (layer 1: base of its inner couplings, mid with the shell's).
template <class Mixed, class Base, class Mid>
void layer_cuts(const Cone& c, const ShellPlanner& sp, const ShellCone& q, int32_t p, int32_t cut_min, Mixed& mixed,
                Base& base, Mid& mid) {
    const int32_t *eb = sp.eb.data() + q.edge, *ew = sp.ew.data() + q.edge;
    double w_all = 0.0;
    for (int32_t e = 0; e < q.n_edges; ++e) w_all += ew[e];
    for (int l = 1; l <= p; ++l) mixed[l] = c.nd[p - l];
    for (int l = 2; l <= p; ++l) {
        int32_t cmin = 0;
        double wl = 0.0;
        for (int32_t e = 0; e < q.n_edges; ++e)
            if (eb[e] < mixed[l - 1]) {
                cmin += std::min(ew[e], 0);
                wl += ew[e];
            }
        base[l] = static_cast<int16_t>(cmin - cut_min);
        mid[l] = static_cast<float>(0.5 * wl - cut_min);
    }
    base[1] = base[2];
    mid[1] = static_cast<float>(0.5 * (w_all - q.w_leaf) - cut_min);
}

// Where the leaves of a cone's shape stand (16 entries, shared by the shape's cones); wz: largest coupling.
int32_t place_leaves(const ShellPlanner& sp, const ShellCone& q, std::vector<int32_t>& at, std::vector<ZLeaf>& out, int32_t& wz) {
    if (!q.zmask) return 0;
    if (at.size() <= static_cast<size_t>(q.shape)) at.resize(static_cast<size_t>(q.shape) + 1, -1);
    int32_t& a = at[static_cast<size_t>(q.shape)];
    if (a < 0) {
        a = static_cast<int32_t>(out.size());
        out.resize(out.size() + 16, ZLeaf{});
        const ShellLeaves* L = sp.leaves(q.shape);
        for (int i = 0; i < q.kin; ++i)
            for (int j = 0; j < ZL_W; ++j) {
                out[static_cast<size_t>(a + i)].w[j] = L[i].w[j];
                out[static_cast<size_t>(a + i)].m[j] = L[i].m[j];
                wz = std::max<int32_t>(wz, L[i].w[j]);
            }
    }
    return a;
}

// Fills P->in_groups and the descriptors for the orbits in ord; their edges are appended to ea, eb, ew.
void build_inner(qaoa_plan_s* P, std::vector<int64_t>& ord, const std::vector<char>& member, std::vector<int32_t>& ea, std::vector<int32_t>& eb,
                 std::vector<int32_t>& ew, InnerHost& in) {
    const HostPlan& hp = P->hp;
    const int32_t p = hp.p;
    const bool by_k = P->opt.profile || P->opt.tune == 1;
    P->in_groups.clear();
    P->in_bands.clear();
    for (auto& list : P->in_rest) list.clear();
    P->in_serial.clear();
    P->n_in_cones = 0;
    P->in_inst.clear();
    P->tr_inst.clear();
    P->in_max_k = 0;   // build_wide adds its own
    P->wz = 0;
    in.band.assign(hp.cones.size(), 0);
    if (ord.empty()) return;
    auto wh_of = [&](int64_t m) {
        return !member.empty() && member[static_cast<size_t>(m)] != 0 ? wh_class(hp.cones[static_cast<size_t>(m)].k) : 0;
    };
    in.cones.reserve(ord.size());
    ShellPlanner shells(p, p == 2, hp.realw);
    std::vector<ShellCone> sc;
    {
        std::vector<const Cone*> list_of(ord.size());
        for (size_t i = 0; i < ord.size(); ++i) list_of[i] = &hp.cones[static_cast<size_t>(ord[i])];
        std::vector<ShellCone> raw;
        shells.add(list_of, raw);
        shells.list();
        std::vector<std::pair<uint32_t, int32_t>> by(ord.size());   // class, place in ord
        for (size_t i = 0; i < by.size(); ++i) {
            const ShellCone& q = raw[i];
            const Cone& c = *list_of[i];
            const uint32_t k = by_k ? static_cast<uint32_t>(c.k) : 0u, wh = static_cast<uint32_t>(wh_of(ord[i]));
            const uint32_t rounds = q.tree ? 0u : shell_rounds(shells, q);
            const int band = in_band(P, c, q.tree, rounds);
            in.band[static_cast<size_t>(ord[i])] = static_cast<char>(band);
            if (band) {
                auto& all = P->in_bands;
                auto at = std::find_if(all.begin(), all.end(), [&](const qaoa_plan_s::Band& b) {
                    return b.K == c.k && b.wh == static_cast<int>(wh);
                });
                if (at == all.end()) at = all.insert(all.end(), {band, static_cast<int>(wh), c.k, 0, 0});
                at->count += 1;
                at->rounds = std::max(at->rounds, static_cast<int32_t>(rounds));
            }
            by[i] = {static_cast<uint32_t>(q.kin) << 12 | k << 6 | wh << 2 | (q.tree ? 2u : 0u) | (q.zmask ? 1u : 0u),
                     static_cast<int32_t>(i)};
        }
        std::sort(by.begin(), by.end());
        std::vector<int64_t> sorted(ord.size());
        sc.resize(ord.size());
        for (size_t i = 0; i < by.size(); ++i) {
            sorted[i] = ord[static_cast<size_t>(by[i].second)];
            sc[i] = raw[static_cast<size_t>(by[i].second)];
        }
        ord.swap(sorted);
    }
    const int64_t edge0 = static_cast<int64_t>(ea.size());
    ea.insert(ea.end(), shells.ea.begin(), shells.ea.end());
    eb.insert(eb.end(), shells.eb.begin(), shells.eb.end());
    ew.insert(ew.end(), shells.ew.begin(), shells.ew.end());
    std::vector<int32_t> leaf_at;
    std::vector<int32_t> type_of(SH_CODES, -1);   // of branches with a code
    auto leaf = [&](double w, int m) { in.leaf2.push_back({w, m, 0}); };
    auto type = [&](double w, int32_t first) {
        in.types.push_back({w, first, static_cast<int32_t>(in.leaf2.size()) - first});
        return static_cast<int32_t>(in.types.size() - 1);
    };
    auto branch_type = [&](const ShellBranch& b) {
        const int32_t first = static_cast<int32_t>(in.leaf2.size());
        if (b.code < 0) {
            for (int i = 0; i < b.n_leaf; ++i) leaf(shells.leaf_w[static_cast<size_t>(b.leaf + i)], 1);
            return type(b.w, first);
        }
        int32_t& t = type_of[static_cast<size_t>(b.code)];
        if (t < 0) {
            for (int x = 1, r = b.code % 343; x <= 3; ++x, r /= 7)
                if (r % 7) leaf(x, r % 7);
            t = type(b.w, first);
        }
        return t;
    };
    // sides of equal branches are one where all of them have a code (the first 64 kinds)
    std::vector<std::array<int16_t, 8>> kinds;
    std::vector<int32_t> kind_side;
    auto side = [&](int32_t first, int n) {
        std::array<int16_t, 8> key;
        key.fill(-1);
        bool coded = true;
        for (int i = 0; i < n; ++i) {
            key[static_cast<size_t>(i)] = shells.branches[static_cast<size_t>(first + i)].code;
            coded = coded && key[static_cast<size_t>(i)] >= 0;
        }
        std::sort(key.begin(), key.begin() + n);
        size_t k = 0;
        while (coded && k < kinds.size() && kinds[k] != key) ++k;
        if (coded && k < kinds.size()) return kind_side[k];
        const int32_t s = static_cast<int32_t>(in.sides.size());
        in.sides.push_back({static_cast<int32_t>(in.branch.size()), n});
        for (int i = 0; i < n; ++i) {
            ShellBranch b = shells.branches[static_cast<size_t>(first + i)];
            if (coded) {
                b.code = key[static_cast<size_t>(i)];
                b.w = b.code / 343 - 3;
            }
            in.branch.push_back(branch_type(b));
        }
        if (coded && kinds.size() < 64) {
            kinds.push_back(key);
            kind_side.push_back(s);
        }
        return s;
    };
    // a group of in_groups continues where its key does
    auto group = [&](const qaoa_plan_s::InGroup& want) -> qaoa_plan_s::InGroup& {
        auto key = [](const qaoa_plan_s::InGroup& g) { return std::tie(g.kin, g.K, g.wh, g.tree, g.signs); };
        if (P->in_groups.empty() || key(P->in_groups.back()) != key(want)) P->in_groups.push_back(want);
        return P->in_groups.back();
    };
    std::vector<int32_t> listed_at;   // first entry of each shape's list, -1: not placed yet
    std::vector<uint32_t> rounds;     // of in.cones
    rounds.reserve(ord.size());
    for (size_t i = 0; i < ord.size(); ++i) {
        const int64_t m = ord[i];
        const Cone& c = hp.cones[m];
        const ShellCone& q = sc[i];
        if (q.tree) {
            D2Cone d{static_cast<int32_t>(m), 0, side(q.br, q.nu), side(q.br + q.nu, q.nv)};
            ShellBranch edge;   // without leaves
            edge.w = q.w_uv;
            if (!hp.realw && std::abs(q.w_uv) <= 3.0) edge.code = static_cast<int16_t>((static_cast<int>(q.w_uv) + 3) * 343);
            d.edge = branch_type(edge);
            qaoa_plan_s::InGroup want{};
            want.K = by_k ? c.k : 0;
            want.wh = wh_of(m);
            want.tree = true;
            want.first = static_cast<int64_t>(in.tr.size());
            group(want).count += 1;
            P->in_max_k = std::max(P->in_max_k, c.k);
            P->tr_inst.push_back(c.inst);
            in.tr.push_back(d);
            continue;
        }
        const uint32_t cpw = shell_at_once(q);
        ConeIn d{};
        d.orbit = static_cast<int32_t>(m);
        d.inst = c.inst;
        d.kin = q.kin;
        layer_cuts(c, shells, q, p, hp.cut_min, d.mixed, d.base, d.mid);
        d.shell_norm = std::ldexp(1.0, -(c.k - q.kin - q.n_leaf));
        d.nc = q.nc;
        d.cfg_off = -1;
        d.zmask = q.zmask;
        d.z_off = place_leaves(shells, q, leaf_at, in.leaf, P->wz);
        uint32_t runs = q.runs();
        if (const std::vector<ShellCfg>* list = shells.configurations(q.shape)) {
            if (listed_at.size() <= static_cast<size_t>(q.shape)) listed_at.resize(static_cast<size_t>(q.shape) + 1, -1);
            int32_t& at = listed_at[static_cast<size_t>(q.shape)];
            d.n_cfg = static_cast<uint32_t>((list->size() + cpw - 1) / cpw * cpw);   // whole rounds
            if (at < 0) {
                at = static_cast<int32_t>(in.cfg.size());
                for (uint32_t e = 0; e < d.n_cfg; ++e) {
                    const ShellCfg& x = (*list)[std::min<size_t>(e, list->size() - 1)];
                    CfgList y{};
                    std::copy_n(x.h, 8, y.h);
                    y.c0 = x.c0;
                    y.z = x.z;
                    y.w = e < list->size() ? x.w : 0.0;
                    in.cfg.push_back(y);
                }
            }
            d.cfg_off = at;
            runs = d.n_cfg;
        } else {   // decoded where they are used
            d.grp_off = static_cast<int32_t>(in.grp.size());
            const std::vector<ShellGroup>& groups = shells.groups(q.shape);
            d.n_grp = static_cast<int32_t>(groups.size());
            for (const ShellGroup& g : groups) {
                GrpIn y{};
                y.m = g.m;
                y.wsum = g.wsum;
                std::copy_n(g.h, 8, y.h);
                in.grp.push_back(y);
            }
        }
        rounds.push_back((runs + cpw - 1) / cpw);
        d.tab_off = static_cast<int32_t>(in.tab_units);
        in.tab_units += (p - 1) * std::max<int64_t>(1, (int64_t{1} << q.kin) / 16);
        d.edge_off = static_cast<int32_t>(edge0 + q.edge);
        d.n_edges = q.n_edges;
        qaoa_plan_s::InGroup want{};
        want.kin = q.kin;
        want.K = by_k ? c.k : 0;
        want.wh = wh_of(m);
        want.signs = q.zmask != 0;
        want.first = static_cast<int64_t>(in.cones.size());
        group(want).count += 1;
        P->in_max_k = std::max(P->in_max_k, c.k);
        P->in_inst.push_back(c.inst);
        in.cones.push_back(d);
    }
    // workgroups and segments of a class whose units are set
    auto place = [&](qaoa_plan_s::InGroup& g) {
        const int64_t ch = g.chunks;
        std::vector<int32_t> unit{0}, inst;   // segments of one instance
        for (int64_t i = 0; i < g.count; ++i) {
            const int32_t j = (g.tree ? P->tr_inst : P->in_inst)[static_cast<size_t>(g.first + i)];
            if (inst.empty() || inst.back() != j) {
                if (!inst.empty()) unit.push_back(static_cast<int32_t>(i * ch));
                inst.push_back(j);
            }
        }
        unit.push_back(static_cast<int32_t>(g.count * ch));
        g.n_seg = static_cast<int32_t>(inst.size());
        for (int j = 0; j < 4; ++j) {
            const int32_t per = (g.tree ? 256 : 4) << j;   // a tree per thread
            int32_t b = 0;
            std::vector<int32_t> blk;
            for (int32_t q = 0; q < g.n_seg; ++q) {
                blk.push_back(b);
                b += (unit[q + 1] - unit[q] + per - 1) / per;
            }
            blk.push_back(b);
            g.blocks[j] = b;
            g.seg[j] = static_cast<int64_t>(in.seg.size());
            if (g.n_seg > 1) {
                in.seg.insert(in.seg.end(), unit.begin(), unit.end());
                in.seg.insert(in.seg.end(), blk.begin(), blk.end());
                in.seg.insert(in.seg.end(), inst.begin(), inst.end());
            }
        }
    };
    for (auto& g : P->in_groups) {
        // Units of work: a cone's rounds in parts of 8, of 2 where that leaves a point with fewer than
        // 1024 units (latency: the 18-qubit cone of a torus at 32 points 42 -> 24 us), at most 2^15
        // of them.  Set by the plan alone, so that a term's sum in this form is the same whatever the
        // number of points.  Classes of cones that fit the allocation-free call (k_lds_max qubits: 16
        // rounds at most) stay whole, as parts need room for their sums.
        uint32_t most = 1;
        int32_t max_k = 0;
        for (int64_t i = g.first; i < g.first + g.count && !g.tree; ++i) {
            most = std::max(most, rounds[static_cast<size_t>(i)]);
            max_k = std::max(max_k, hp.cones[static_cast<size_t>(in.cones[static_cast<size_t>(i)].orbit)].k);
        }
        int64_t ch = 1;
        if (max_k > P->opt.k_lds_max) {
            ch = (most + IN_ROUNDS - 1) / IN_ROUNDS;
            if (ch * g.count < 1024) ch = std::min<int64_t>((most + 1) / 2, std::max<int64_t>(ch, 1024 / g.count));
        }
        ch = std::min(ch, std::max<int64_t>(1, (int64_t{1} << 15) / g.count));
        g.chunks = static_cast<int32_t>(ch);
        place(g);
        for (int64_t i = g.first; i < g.first + g.count && !g.tree; ++i)
            if (in.band[static_cast<size_t>(in.cones[static_cast<size_t>(i)].orbit)] != 3)
                g.rounds = std::max(g.rounds, static_cast<int32_t>((rounds[static_cast<size_t>(i)] + ch - 1) / ch));
        for (int j = 0; j < 2 && !g.tree; ++j) {
            int32_t n = 0;   // of the instance
            for (int64_t i = g.first; i < g.first + g.count; ++i) {
                const size_t at = static_cast<size_t>(i);
                if (i > g.first && P->in_inst[at] != P->in_inst[at - 1]) n = 0;
                const int band = in.band[static_cast<size_t>(in.cones[at].orbit)];
                if (band >= 1 && band <= j + 1 && n++ % 4 == 0) g.small[j] += 1;
            }
        }
    }
    P->n_in_cones = static_cast<int64_t>(in.cones.size());
    for (const auto& b : P->in_bands)
        if (b.band == 3 && std::find(P->in_serial.begin(), P->in_serial.end(), b.K) == P->in_serial.end())
            P->in_serial.push_back(b.K);
    auto most = [&](int K) {
        int32_t n = 0;
        for (const auto& b : P->in_bands) n = std::max(n, b.K == K ? b.rounds : 0);
        return n;
    };
    std::sort(P->in_serial.begin(), P->in_serial.end(), [&](int x, int y) { return std::make_pair(-most(x), x) < std::make_pair(-most(y), y); });
    for (int rest = 0; rest < 2 + static_cast<int>(P->in_serial.size()) && !P->in_bands.empty(); ++rest) {
        uint32_t sizes = rest == 0 ? (1u << 10) - 1 : rest == 1 ? (1u << 11) - 1 : 0;   // that leave
        for (int j = 0; j < rest - 1; ++j) sizes |= 1u << P->in_serial[static_cast<size_t>(j)];
        for (const auto& all : P->in_groups) {
            if (all.tree) {
                P->in_rest[rest].push_back(all);
                continue;
            }
            auto stays = [&](int64_t i) {
                const size_t m = static_cast<size_t>(in.cones[static_cast<size_t>(i)].orbit);
                return in.band[m] == 0 || !((sizes >> hp.cones[m].k) & 1u);
            };
            qaoa_plan_s::InGroup g = all;
            g.count = 0;
            for (int64_t i = all.first; i < all.first + all.count; ++i) g.count += stays(i);
            if (g.count == 0) continue;
            if (g.count < all.count) {   // its units are those of the whole class, and so a term's sum
                g.first = static_cast<int64_t>(in.cones.size());
                for (int64_t i = all.first; i < all.first + all.count; ++i)
                    if (stays(i)) {
                        const ConeIn copy = in.cones[static_cast<size_t>(i)];
                        in.cones.push_back(copy);
                        P->in_inst.push_back(P->in_inst[static_cast<size_t>(i)]);
                    }
                place(g);
            }
            P->in_rest[rest].push_back(g);
        }
    }
}

// The units of a plan whose calls are one launch (inner_point.hip): one instance, all cones on their
// inner qubits with listed configurations, and at most 16 units and orbits.  Up to there one
// compute unit holds a point's waves at once; the 18-qubit cone of a torus, 19 units of two rounds
// each, would run them one after the other where the separate launches spread them over five.
// Beyond four units few points are spread as well (IN_SPREAD), and many at p = 2 (enqueue).  Up to
// four there is no line at any number of points: a class's launch gives a point's few units a
// workgroup of their own too, and leaves its other waves idle (energy and gradient of C_10000(1,2) at
// p = 2, 1, 256, 2048 and 16384 points: 18.8, 17.9, 36, 191 us in separate launches, 13.6, 13.3, 22,
// 109 here; rings at p = 3 .. 5, 1 point: 16, 19, 42 us and 13, 18, 41; 16384 points: 218, 309, 778 us
// and 101, 152, 379).
void build_point(qaoa_plan_s* P, const InnerHost& in) {
    P->in_point = InPoint{};
    P->in_parts = InPointSum{};
    const size_t M = P->hp.cones.size();
    P->d2_point = false;
    if (P->hp.n_inst != 1 || M > D2_POINT || static_cast<size_t>(P->n_in_cones) + in.tr.size() != M || !P->wh_groups.empty() || P->opt.profile ||
        P->opt.tune != 0 || P->opt.one_cone_at_a_time)
        return;
    if (in.cones.empty()) {   // trees, in orbit order
        P->d2_point = P->in_groups.size() == 1;
        return;
    }
    if (M > IN_POINT) return;
    const size_t rows = static_cast<size_t>(3 + P->hp.p) * (P->hp.cut_max - P->hp.cut_min + 1) * sizeof(float2) +
                        static_cast<size_t>(P->wz + 1) * sizeof(double2);
    const size_t sums = P->hp.p > 2 ? static_cast<size_t>(in_point_waves(true, 0)) * (2 * P->hp.p + 1) * 512 : 0;
    // too many units for a workgroup per point: units first, then all sums
    auto parts = [&]() {
        InPointSum& s = P->in_parts;
        if (!in.tr.empty()) return;
        for (const auto& g : P->in_groups)
            for (int64_t i = 0; i < g.count; ++i) {
                InPointSum::Cone& c = s.c[s.n++];
                c.units = static_cast<int32_t>(g.count * g.chunks);
                c.unit0 = static_cast<int32_t>(i * g.chunks);
                c.chunks = g.chunks;
                c.orbit = in.cones[static_cast<size_t>(g.first + i)].orbit;
            }
    };
    if (rows + sums > IN_POINT_LDS) return parts();
    InPoint q{};
    auto u16 = [](int64_t x) { return static_cast<uint16_t>(x); };
    for (const auto& g : P->in_groups)
        for (int64_t i = g.first; i < g.first + g.count; ++i) {
            if (q.n_part + g.chunks > IN_POINT || q.n + g.chunks > IN_POINT) return parts();
            if (g.tree) {
                if (i == g.first)
                    q.unit[q.n++] = {u16(i), 0, 1, u16(q.n_part), 0, static_cast<uint8_t>(g.count)};
                q.part[q.n_part++] = {1, u16(in.tr[static_cast<size_t>(i)].orbit)};
                continue;
            }
            const ConeIn& c = in.cones[static_cast<size_t>(i)];
            if (c.cfg_off < 0) return parts();
            for (int32_t ch = 0; ch < g.chunks; ++ch) {
                q.unit[q.n++] = {u16(i), u16(ch), u16(g.chunks), u16(q.n_part), static_cast<uint8_t>(c.kin), 0};
                q.part[q.n_part++] = {u16(g.chunks), u16(c.orbit)};
            }
        }
    P->in_point = q;
    if (q.n > 4) parts();   // for few points
}

// Plans whose cones of 10 qubits never run whole (choose_forms).
bool ten_stay(const qaoa_plan_s* P) { return P->in_point.n > 0 && P->in_point.n <= 4; }

struct WideHost {
    std::vector<ConeWd> cones;
    std::vector<UnitWd> units;
    std::vector<GrpWd> grp;
    std::vector<CfgWd> cfg;
    std::vector<ZLeaf> leaf;
    int64_t tab_bytes = 0;
    bool too_many = false;   // units: more than 32-bit integers index
};

// Fills P->wd_groups and the descriptors for the orbits in ord (wide.hpp); their edges are appended.
// A cone's units depend on the cone alone, so its sums are the same in every plan and call.
void build_wide(qaoa_plan_s* P, std::vector<int64_t>& ord, std::vector<int32_t>& ea, std::vector<int32_t>& eb,
                std::vector<int32_t>& ew, WideHost& w) {
    const HostPlan& hp = P->hp;
    const int32_t p = hp.p;
    P->wd_groups.clear();
    P->wd_units.clear();
    P->wd_all_units = 0;
    P->wd_most_units = 0;
    P->wd_rows = 1;
    if (ord.empty()) return;
    const bool by_k = P->opt.profile != 0;
    std::stable_sort(ord.begin(), ord.end(), [&](int64_t a, int64_t b) {
        const Cone &x = hp.cones[static_cast<size_t>(a)], &y = hp.cones[static_cast<size_t>(b)];
        if (x.nd[p - 1] != y.nd[p - 1]) return x.nd[p - 1] < y.nd[p - 1];
        return by_k && x.k < y.k;
    });
    ShellPlanner shells(p);
    std::vector<ShellCone> sc;
    std::vector<const Cone*> list_of(ord.size());
    for (size_t i = 0; i < ord.size(); ++i) list_of[i] = &hp.cones[static_cast<size_t>(ord[i])];
    shells.add(list_of, sc);
    shells.list();
    const int64_t edge0 = static_cast<int64_t>(ea.size());
    ea.insert(ea.end(), shells.ea.begin(), shells.ea.end());
    eb.insert(eb.end(), shells.eb.begin(), shells.eb.end());
    ew.insert(ew.end(), shells.ew.begin(), shells.ew.end());
    std::vector<int32_t> leaf_at;
    std::vector<int32_t> listed_at;   // first entry of each shape's list, -1: not placed yet
    for (size_t i = 0; i < ord.size(); ++i) {
        const Cone& c = hp.cones[static_cast<size_t>(ord[i])];
        const ShellCone& q = sc[i];
        ConeWd d{};
        d.orbit = static_cast<int32_t>(ord[i]);
        d.inst = c.inst;
        d.kin = q.kin;
        d.nc = q.nc;
        d.cut_min = c.cut_min;
        d.n_rows = c.cut_max - c.cut_min + 1;
        P->wd_rows = std::max(P->wd_rows, d.n_rows);
        layer_cuts(c, shells, q, p, c.cut_min, d.mixed, d.base, d.mid);
        d.shell_norm = std::ldexp(1.0, -(c.k - q.kin - q.n_leaf));
        d.cfg_off = -1;
        d.zmask = q.zmask;
        d.z_off = place_leaves(shells, q, leaf_at, w.leaf, P->wz);
        d.n_cfg = q.runs();
        if (const std::vector<ShellCfg>* list = shells.configurations(q.shape)) {
            if (listed_at.size() <= static_cast<size_t>(q.shape)) listed_at.resize(static_cast<size_t>(q.shape) + 1, -1);
            int32_t& at = listed_at[static_cast<size_t>(q.shape)];
            if (at < 0) {
                at = static_cast<int32_t>(w.cfg.size());
                for (const ShellCfg& x : *list) {
                    CfgWd y{};
                    std::copy_n(x.h, SH_H, y.h);
                    y.c0 = x.c0;
                    y.z = x.z;
                    y.w = x.w;
                    w.cfg.push_back(y);
                }
            }
            d.cfg_off = at;
            d.n_cfg = static_cast<uint32_t>(list->size());
        } else {
            d.grp_off = static_cast<int32_t>(w.grp.size());
            const std::vector<ShellGroup>& groups = shells.groups(q.shape);
            d.n_grp = static_cast<int32_t>(groups.size());
            for (const ShellGroup& g : groups) {
                GrpWd y{};
                y.m = g.m;
                y.wsum = g.wsum;
                std::copy_n(g.h, SH_H, y.h);
                w.grp.push_back(y);
            }
        }
        d.tab_off = w.tab_bytes;
        w.tab_bytes += static_cast<int64_t>(p - 1) << q.kin;
        d.edge_off = static_cast<int32_t>(edge0 + q.edge);
        d.n_edges = q.n_edges;
        const int kk = by_k ? c.k : 0;
        if (P->wd_groups.empty() || P->wd_groups.back().kin != q.kin || P->wd_groups.back().K != kk)
            P->wd_groups.push_back({q.kin, kk, static_cast<int64_t>(w.units.size()), 0});
        d.first_unit = static_cast<int32_t>(w.units.size());
        for (uint32_t c0 = 0; c0 < d.n_cfg; c0 += WD_CFG)
            w.units.push_back({static_cast<int32_t>(i), c0, std::min<uint32_t>(d.n_cfg, c0 + WD_CFG)});
        if (w.units.size() > static_cast<size_t>(INT32_MAX)) {
            w.too_many = true;
            return;
        }
        d.n_units = static_cast<int32_t>(w.units.size()) - d.first_unit;
        P->wd_most_units = std::max<int64_t>(P->wd_most_units, d.n_units);
        P->wd_groups.back().count += d.n_units;
        P->wd_units.emplace_back(d.first_unit, d.n_units);
        P->in_max_k = std::max(P->in_max_k, c.k);
        w.cones.push_back(d);
    }
    P->wd_all_units = static_cast<int64_t>(w.units.size());
}

qaoa_status ensure_device(qaoa_plan_s* P, std::string& msg) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) {
        msg = std::string("no HIP device: ") + hipGetErrorString(e);
        return QAOA_EHIP;
    }
    if (P->dev_ready) {
        if (dev != P->device) {
            msg = "plan was uploaded to device " + std::to_string(P->device) + ", current device is " + std::to_string(dev);
            return QAOA_EINVAL;
        }
        return QAOA_OK;
    }
    const HostPlan& hp = P->hp;
    const int64_t Mall = static_cast<int64_t>(hp.cones.size());
    // workgroup-resident cones (k <= k_lds_max), grouped by K; larger cones go to the
    // HBM-resident passes, grouped by k
    std::vector<int64_t> ord, hord;
    const bool d1 = depth1_closed(P);
    P->max_k = 0;
    for (const Cone& c : hp.cones) P->max_k = std::max(P->max_k, c.k);
    WholeHost wh;
    build_whole(P, wh);
    auto member = [&](int64_t m) { return !wh.member.empty() && wh.member[static_cast<size_t>(m)]; };
    std::vector<int64_t> d1ord, inord, wdord;
    std::vector<char> inner_of(static_cast<size_t>(Mall), 0);
    for (int64_t m = 0; m < Mall && !d1; ++m)
        if (!wide_cone(P, hp.cones[m]) && inner_cone(P, hp.cones[m])) {
            inner_of[static_cast<size_t>(m)] = 1;
            inord.push_back(m);
        }
    std::vector<int32_t> ea, eb, ew;
    InnerHost in;
    build_inner(P, inord, wh.member, ea, eb, ew, in);
    build_point(P, in);
    if (ten_stay(P))   // no need of their other form
        for (int64_t m : inord)
            if (hp.cones[static_cast<size_t>(m)].k == 10) in.band[static_cast<size_t>(m)] = 0;
    for (int64_t m = 0; m < Mall; ++m) {
        const bool small = hp.cones[m].k <= P->opt.k_lds_max, inner = inner_of[static_cast<size_t>(m)] != 0;
        if (!d1 && !inner && wide_cone(P, hp.cones[m])) {
            wdord.push_back(m);
            continue;
        }
        // (the tuner compares both kernels; a group's state reads its representative's cut table)
        if (inner && !(P->opt.tune == 1 && small) && !member(m) && in.band[static_cast<size_t>(m)] == 0) continue;
        (d1 ? d1ord : small ? ord : hord).push_back(m);
    }
    auto part_of = [&](int64_t m) {   // Group::n_part; tune = 1: cones in both forms first
        const bool inner = inner_of[static_cast<size_t>(m)] != 0, both = in.band[static_cast<size_t>(m)] != 0;
        if (P->opt.tune == 1) return inner ? 3 : 4;
        return member(m) ? (both ? 1 : inner ? 0 : 2) : both ? 3 : 4;
    };
    std::stable_sort(ord.begin(), ord.end(), [&](int64_t a, int64_t b) {
        const Cone &x = hp.cones[a], &y = hp.cones[b];
        return x.k != y.k ? x.k < y.k : part_of(a) < part_of(b);
    });
    std::stable_sort(hord.begin(), hord.end(), [&](int64_t a, int64_t b) { return hp.cones[a].k < hp.cones[b].k; });
    const int64_t M = static_cast<int64_t>(ord.size());
    std::vector<ConeDev> cd(M);
    std::vector<double> ewd(hp.realw ? ea.size() : 0, 0.0);   // real weights (plans with real weights only)
    int64_t cut_bytes = 0;
    P->lds_groups.clear();
    for (int64_t s = 0; s < M; ++s) {
        const Cone& c = hp.cones[ord[s]];
        ConeDev& d = cd[s];
        d.orbit = static_cast<int32_t>(ord[s]);
        d.k = c.k;
        d.edge_off = static_cast<int32_t>(ea.size());
        d.n_edges = static_cast<int32_t>(c.ea.size());
        d.inst = c.inst;
        d.c0 = 0.f;
        d.pad_ = 0;
        if (hp.realw) {
            // float table of C(x) - c0 over the stored half; cut_off counts floats
            d.cut_off = cut_bytes / 4;
            d.cut_shift = 0;
            d.cut_min = 0;
            d.cut_range = 1;
            d.c0 = static_cast<float>(0.5 * (c.cf_min + c.cf_max));
            cut_bytes += 4 * std::max<int64_t>(int64_t{1} << (c.k >= 3 ? c.k - 1 : c.k), 4);
            ewd.insert(ewd.end(), c.wf.begin(), c.wf.end());
        } else {
            d.cut_off = cut_bytes;
            d.cut_shift = c.cut_min - hp.cut_min;
            d.cut_min = c.cut_min;
            d.cut_range = c.cut_max - c.cut_min + 1;
            cut_bytes += std::max<int64_t>(int64_t{1} << c.k, 16);
        }
        ea.insert(ea.end(), c.ea.begin(), c.ea.end());
        eb.insert(eb.end(), c.eb.begin(), c.eb.end());
        ew.insert(ew.end(), c.ew.begin(), c.ew.end());
        if (P->lds_groups.empty() || P->lds_groups.back().K != c.k) P->lds_groups.push_back({c.k, s, 0, 1});
        P->lds_groups.back().count += 1;
        P->lds_groups.back().n_part[part_of(ord[s])] += 1;
        if (P->opt.tune == 1 && inner_of[static_cast<size_t>(ord[s])]) P->lds_groups.back().n_in += 1;
        P->lds_groups.back().rowcap = std::max(P->lds_groups.back().rowcap, d.cut_range);
    }
    WideHost wd;
    build_wide(P, wdord, ea, eb, ew, wd);
    if (wd.too_many) {
        msg = "the plan's cones take more than 2^31 - 1 units of work; descriptors index them with 32-bit integers";
        return QAOA_EINVAL;
    }
    // depth-1 cones: the couplings of the edge's two ends
    std::vector<ConeD1> dc(d1ord.size());
    std::vector<double2> dw;
    P->d1_groups.clear();
    const bool d1_by_k = P->opt.profile || P->opt.one_cone_at_a_time;
    if (d1_by_k)
        std::stable_sort(d1ord.begin(), d1ord.end(), [&](int64_t a, int64_t b) { return hp.cones[a].k < hp.cones[b].k; });
    for (size_t s = 0; s < d1ord.size(); ++s) {
        const Cone& c = hp.cones[d1ord[s]];
        ConeD1& d = dc[s];
        if (dw.size() > static_cast<size_t>(INT32_MAX) - 32) {
            msg = "the plan's cones hold more than 2^31 - 1 neighbours; descriptors index them with 32-bit integers";
            return QAOA_EINVAL;
        }
        d = {static_cast<int32_t>(d1ord[s]), c.inst, static_cast<int32_t>(dw.size()), c.k - 2, 0.0};
        dw.resize(dw.size() + static_cast<size_t>(c.k - 2), double2{0.0, 0.0});
        for (size_t e = 0; e < c.ea.size(); ++e) {
            if (c.ea[e] > 1) continue;   // couplings between neighbours have no part in the term
            const double w = hp.realw ? c.wf[e] : static_cast<double>(c.ew[e]);
            if (c.eb[e] == 1) {
                d.wuv = w;
            } else {
                double2& x = dw[static_cast<size_t>(d.off + c.eb[e] - 2)];
                (c.ea[e] == 0 ? x.x : x.y) = w;
            }
        }
        const int kk = d1_by_k ? c.k : 0;
        if (P->d1_groups.empty() || P->d1_groups.back().K != kk)
            P->d1_groups.push_back({kk, static_cast<int64_t>(s), 0, 1});
        P->d1_groups.back().count += 1;
    }
    // HBM-class descriptors; their edges follow the workgroup-resident ones
    std::vector<ConeHbm> hc(hord.size());
    int64_t tt_bytes = 0;
    int max_groups = 1;
    P->hbm_groups.clear();
    for (size_t s = 0; s < hord.size(); ++s) {
        const Cone& c = hp.cones[hord[s]];
        ConeHbm& d = hc[s];
        std::memset(&d, 0, sizeof(d));
        d.orbit = static_cast<int32_t>(hord[s]);
        d.k = c.k;
        d.edge_off = static_cast<int32_t>(ea.size());
        d.n_edges = static_cast<int32_t>(c.ea.size());
        d.cut_min = c.cut_min;
        d.cut_range = c.cut_max - c.cut_min + 1;
        d.cut_shift = c.cut_min - hp.cut_min;
        d.inst = c.inst;
        d.c0 = static_cast<float>(0.5 * (c.cf_min + c.cf_max));
        d.n_groups = hbm_groups_of(c.k - 1);
        max_groups = std::max(max_groups, d.n_groups);
        for (int g = 0; g < d.n_groups; ++g) {
            // tile bits of group g; C_tt ranges over the edges with both ends inside
            std::vector<char> in(32, 0);
            for (int i = 0; i < 13; ++i) in[hbm_group_global_bit(c.k - 1, g, i)] = 1;
            int32_t tmin = 0, tmax = 0;
            for (size_t e = 0; e < c.ea.size(); ++e)
                if (in[c.ea[e]] && in[c.eb[e]]) (c.ew[e] < 0 ? tmin : tmax) += c.ew[e];
            d.tt_min[g] = tmin;
            // byte table of 2^13 entries, or (real weights) floats: tt_off then counts floats
            d.tt_off[g] = hp.realw ? tt_bytes / 4 : tt_bytes;
            tt_bytes += hp.realw ? 4 * 8192 : 8192;
        }
        ea.insert(ea.end(), c.ea.begin(), c.ea.end());
        eb.insert(eb.end(), c.eb.begin(), c.eb.end());
        ew.insert(ew.end(), c.ew.begin(), c.ew.end());
        if (hp.realw) ewd.insert(ewd.end(), c.wf.begin(), c.wf.end());
        if (P->hbm_groups.empty() || P->hbm_groups.back().K != c.k)
            P->hbm_groups.push_back({c.k, static_cast<int64_t>(s), 0, 1});
        P->hbm_groups.back().count += 1;
        P->hbm_groups.back().rowcap = std::max(P->hbm_groups.back().rowcap, d.cut_range);
    }
    if (ea.size() > static_cast<size_t>(INT32_MAX) || Mall > INT32_MAX || in.tab_units > INT32_MAX) {
        msg = "the plan's cones hold " + std::to_string(ea.size()) + " edges over " + std::to_string(Mall) +
              " orbits; descriptors index both with 32-bit integers";
        return QAOA_EINVAL;
    }
    // One device allocation holds every resident array: the ones with host data first (one
    // copy), then the cut and C_tt tables, which kernels fill.
    const size_t ne = std::max<size_t>(ea.size(), 1);
    const std::vector<double> ones(hp.inst_delta.size(), 1.0);
    size_t arena = 0;
    auto place = [&](size_t bytes) {
        const size_t o = arena;
        arena += (std::max<size_t>(bytes, 16) + 255) & ~size_t{255};
        return o;
    };
    const size_t o_cones = place(std::max<size_t>(cd.size(), 1) * sizeof(ConeDev));
    const size_t o_W = place(std::max<size_t>(hp.W.size(), 1) * sizeof(double));
    const size_t o_hcones = place(std::max<size_t>(hc.size(), 1) * sizeof(ConeHbm));
    const size_t o_ea = place(ne * sizeof(int32_t));
    const size_t o_eb = place(ne * sizeof(int32_t));
    const size_t o_ew = place(ne * sizeof(int32_t));
    const size_t o_io = place(hp.inst_orbit.size() * sizeof(int64_t));
    const size_t o_id = place(hp.inst_delta.size() * sizeof(double));
    const size_t o_ones = place(ones.size() * sizeof(double));
    const size_t o_ewd = hp.realw ? place(std::max<size_t>(ewd.size(), 1) * sizeof(double)) : 0;
    const size_t o_dc = d1 ? place(dc.size() * sizeof(ConeD1)) : 0;
    const size_t o_dw = d1 ? place(dw.size() * sizeof(double2)) : 0;
    if (!wh.groups.empty()) {   // their representatives' cut tables
        std::vector<int64_t> cut_of(static_cast<size_t>(Mall), 0);
        for (const ConeDev& d : cd) cut_of[static_cast<size_t>(d.orbit)] = d.cut_off;
        for (GroupWh& g : wh.groups) g.cut_off = cut_of[static_cast<size_t>(g.rep)];
    }
    const bool has_wh = !wh.groups.empty();
    const size_t o_wg = has_wh ? place(wh.groups.size() * sizeof(GroupWh)) : 0;
    const size_t o_wm = has_wh ? place(wh.mem.size() * sizeof(MemWh)) : 0;
    const size_t o_ww = has_wh ? place(wh.Wg.size() * sizeof(double)) : 0;
    const bool has_in = !in.cones.empty();
    const size_t o_in = has_in ? place(in.cones.size() * sizeof(ConeIn)) : 0;
    const size_t o_ig = has_in ? place(in.grp.size() * sizeof(GrpIn)) : 0;
    const bool has_wd = !wd.cones.empty();
    const size_t o_dco = has_wd ? place(wd.cones.size() * sizeof(ConeWd)) : 0;
    const size_t o_dun = has_wd ? place(wd.units.size() * sizeof(UnitWd)) : 0;
    const size_t o_dgr = has_wd ? place(wd.grp.size() * sizeof(GrpWd)) : 0;
    const size_t o_dlf = has_wd ? place(wd.leaf.size() * sizeof(ZLeaf)) : 0;
    const size_t o_ilf = has_in ? place(in.leaf.size() * sizeof(ZLeaf)) : 0;
    const size_t o_dcf = has_wd ? place(wd.cfg.size() * sizeof(CfgWd)) : 0;
    const bool has_tr = !in.tr.empty();
    const size_t o_tr = has_tr ? place(in.tr.size() * sizeof(D2Cone)) : 0;
    const size_t o_ts = has_tr ? place(in.sides.size() * sizeof(D2SideDef)) : 0;
    const size_t o_tb = has_tr ? place(in.branch.size() * sizeof(int32_t)) : 0;
    const size_t o_tt2 = has_tr ? place(in.types.size() * sizeof(D2Type)) : 0;
    const size_t o_tl = has_tr ? place(in.leaf2.size() * sizeof(D2Leaf)) : 0;
    const size_t o_ic = has_in ? place(in.cfg.size() * sizeof(CfgList)) : 0;
    const bool has_seg = !in.seg.empty();
    const size_t o_is = has_seg ? place(in.seg.size() * sizeof(int32_t)) : 0;
    const size_t copied = arena;
    const size_t o_wo = has_wh ? place(static_cast<size_t>(wh.obs) * sizeof(double)) : 0;
    const size_t o_dta = has_wd ? place(static_cast<size_t>(wd.tab_bytes)) : 0;
    const size_t o_it = has_in ? place(static_cast<size_t>(in.tab_units) * 16) : 0;
    const size_t o_cut = place(static_cast<size_t>(std::max<int64_t>(cut_bytes, 16)));
    const size_t o_tt = place(static_cast<size_t>(std::max<int64_t>(tt_bytes, 16)));
    {
        // staged in pinned host memory shared by all plans of the process (grown on demand,
        // kept until exit): one fast copy instead of a pageable one (3 MB: 1.1 ms -> ~0.1 ms)
        std::lock_guard<std::mutex> lock(g_stage_mu);
        if (g_stage_cap < copied) {
            if (g_stage) hipHostFree(g_stage);
            g_stage = nullptr;
            g_stage_cap = 0;
            const size_t cap = std::max<size_t>(copied, size_t{4} << 20);
            QCHECK(hipHostMalloc(&g_stage, cap, hipHostMallocPortable));
            g_stage_cap = cap;
        }
        uint8_t* stage = static_cast<uint8_t*>(g_stage);   // the gaps between arrays are never read
        auto put = [&](size_t o, const void* src, size_t bytes) {
            if (bytes) std::memcpy(stage + o, src, bytes);
        };
        put(o_cones, cd.data(), cd.size() * sizeof(ConeDev));
        put(o_W, hp.W.data(), hp.W.size() * sizeof(double));
        put(o_hcones, hc.data(), hc.size() * sizeof(ConeHbm));
        put(o_ea, ea.data(), ea.size() * sizeof(int32_t));
        put(o_eb, eb.data(), eb.size() * sizeof(int32_t));
        put(o_ew, ew.data(), ew.size() * sizeof(int32_t));
        put(o_io, hp.inst_orbit.data(), hp.inst_orbit.size() * sizeof(int64_t));
        put(o_id, hp.inst_delta.data(), hp.inst_delta.size() * sizeof(double));
        put(o_ones, ones.data(), ones.size() * sizeof(double));
        if (hp.realw) put(o_ewd, ewd.data(), ewd.size() * sizeof(double));
        if (has_wh) {
            put(o_wg, wh.groups.data(), wh.groups.size() * sizeof(GroupWh));
            put(o_wm, wh.mem.data(), wh.mem.size() * sizeof(MemWh));
            put(o_ww, wh.Wg.data(), wh.Wg.size() * sizeof(double));
        }
        if (has_tr) {
            put(o_tr, in.tr.data(), in.tr.size() * sizeof(D2Cone));
            put(o_ts, in.sides.data(), in.sides.size() * sizeof(D2SideDef));
            put(o_tb, in.branch.data(), in.branch.size() * sizeof(int32_t));
            put(o_tt2, in.types.data(), in.types.size() * sizeof(D2Type));
            put(o_tl, in.leaf2.data(), in.leaf2.size() * sizeof(D2Leaf));
        }
        if (has_wd) {
            put(o_dco, wd.cones.data(), wd.cones.size() * sizeof(ConeWd));
            put(o_dun, wd.units.data(), wd.units.size() * sizeof(UnitWd));
            put(o_dgr, wd.grp.data(), wd.grp.size() * sizeof(GrpWd));
            put(o_dlf, wd.leaf.data(), wd.leaf.size() * sizeof(ZLeaf));
            put(o_dcf, wd.cfg.data(), wd.cfg.size() * sizeof(CfgWd));
        }
        if (has_in) {
            put(o_in, in.cones.data(), in.cones.size() * sizeof(ConeIn));
            put(o_ig, in.grp.data(), in.grp.size() * sizeof(GrpIn));
            put(o_ilf, in.leaf.data(), in.leaf.size() * sizeof(ZLeaf));
            put(o_ic, in.cfg.data(), in.cfg.size() * sizeof(CfgList));
        }
        if (has_seg) put(o_is, in.seg.data(), in.seg.size() * sizeof(int32_t));
        if (d1) {
            put(o_dc, dc.data(), dc.size() * sizeof(ConeD1));
            put(o_dw, dw.data(), dw.size() * sizeof(double2));
        }
        if (P->d_arena) {   // an earlier first call failed after allocating: start over
            hipFree(P->d_arena);
            P->d_arena = nullptr;
        }
        QCHECK(hipMalloc(&P->d_arena, arena));
        QCHECK(hipMemcpy(P->d_arena, stage, copied, hipMemcpyHostToDevice));
    }
    uint8_t* base = static_cast<uint8_t*>(P->d_arena);
    P->d_cones = reinterpret_cast<ConeDev*>(base + o_cones);
    P->d_W = reinterpret_cast<double*>(base + o_W);
    P->d_hcones = reinterpret_cast<ConeHbm*>(base + o_hcones);
    P->d_ea = reinterpret_cast<int32_t*>(base + o_ea);
    P->d_eb = reinterpret_cast<int32_t*>(base + o_eb);
    P->d_ew = reinterpret_cast<int32_t*>(base + o_ew);
    P->d_inst_orbit = reinterpret_cast<int64_t*>(base + o_io);
    P->d_inst_delta = reinterpret_cast<double*>(base + o_id);
    P->d_ones = reinterpret_cast<double*>(base + o_ones);
    P->d_ewd = hp.realw ? reinterpret_cast<double*>(base + o_ewd) : nullptr;
    P->d_d1 = d1 ? reinterpret_cast<ConeD1*>(base + o_dc) : nullptr;
    P->d_d1w = d1 ? reinterpret_cast<double2*>(base + o_dw) : nullptr;
    P->d_wh = has_wh ? reinterpret_cast<GroupWh*>(base + o_wg) : nullptr;
    P->d_whmem = has_wh ? reinterpret_cast<MemWh*>(base + o_wm) : nullptr;
    P->d_Wg = has_wh ? reinterpret_cast<double*>(base + o_ww) : nullptr;
    P->d_whobs = has_wh ? reinterpret_cast<double*>(base + o_wo) : nullptr;
    P->d_wd = has_wd ? reinterpret_cast<ConeWd*>(base + o_dco) : nullptr;
    P->d_wdunit = has_wd ? reinterpret_cast<UnitWd*>(base + o_dun) : nullptr;
    P->d_wdgrp = has_wd ? reinterpret_cast<GrpWd*>(base + o_dgr) : nullptr;
    P->d_wdleaf = has_wd ? reinterpret_cast<ZLeaf*>(base + o_dlf) : nullptr;
    P->d_wdcfg = has_wd ? reinterpret_cast<CfgWd*>(base + o_dcf) : nullptr;
    P->d_wdtab = has_wd ? base + o_dta : nullptr;
    P->d_in = has_in ? reinterpret_cast<ConeIn*>(base + o_in) : nullptr;
    P->d_ingrp = has_in ? reinterpret_cast<GrpIn*>(base + o_ig) : nullptr;
    P->d_tr = has_tr ? reinterpret_cast<D2Cone*>(base + o_tr) : nullptr;
    P->d_sides = has_tr ? reinterpret_cast<D2SideDef*>(base + o_ts) : nullptr;
    P->n_sides = static_cast<int32_t>(in.sides.size());
    P->d_branch = has_tr ? reinterpret_cast<int32_t*>(base + o_tb) : nullptr;
    P->d_types = has_tr ? reinterpret_cast<D2Type*>(base + o_tt2) : nullptr;
    P->d_leaf2 = has_tr ? reinterpret_cast<D2Leaf*>(base + o_tl) : nullptr;
    P->n_types = static_cast<int32_t>(in.types.size());
    P->d_leaf = has_in ? reinterpret_cast<ZLeaf*>(base + o_ilf) : nullptr;
    P->d_incfg = has_in ? reinterpret_cast<CfgList*>(base + o_ic) : nullptr;
    P->d_inseg = has_seg ? reinterpret_cast<int32_t*>(base + o_is) : nullptr;
    P->d_intab = has_in ? base + o_it : nullptr;
    P->d_cut = base + o_cut;
    P->d_tt = base + o_tt;
    if (d1) {
        // no tables
    } else if (hp.realw) {
        QCHECK(launch_cut_tables_real(P->d_cones, M, P->d_ea, P->d_eb, P->d_ewd, reinterpret_cast<float*>(P->d_cut),
                                      nullptr));
        QCHECK(launch_tt_tables_real(P->d_hcones, static_cast<int64_t>(hc.size()), max_groups, P->d_ea, P->d_eb,
                                     P->d_ewd, reinterpret_cast<float*>(P->d_tt), nullptr));
    } else {
        const PlanTabs tabs = {P->d_cones, P->d_in, P->d_ea, P->d_eb, P->d_ew, P->d_cut, P->d_intab, M, has_in ? P->n_in_cones : 0,
                               hp.p, hp.cut_min, 0, 0};
        QCHECK(launch_plan_tables(tabs, M ? cd.back().k : 0, nullptr));
        QCHECK(launch_tt_tables(P->d_hcones, static_cast<int64_t>(hc.size()), max_groups, P->d_ea, P->d_eb,
                                P->d_ew, P->d_tt, nullptr));
        if (has_wd)
            QCHECK(launch_wide_tables(P->d_wd, static_cast<int64_t>(wd.cones.size()), P->d_ea, P->d_eb, P->d_ew, hp.p,
                                      P->d_wdtab, nullptr));
    }
    for (const auto& g : P->wh_groups)
        QCHECK(launch_whole_obs(P->d_wh + g.first, g.count, P->d_whmem, g.K, P->d_whobs, nullptr));
    QCHECK(hipDeviceSynchronize());
    P->resident_bytes = arena;
    P->device = dev;
    P->dev_ready = true;
    return QAOA_OK;
}

// Events around one kernel group (profiling only).
struct GroupTimer {
    qaoa_plan_s* P;
    hipStream_t st;
    size_t slot = 0;
    bool on;
    GroupTimer(qaoa_plan_s* p, hipStream_t s) : P(p), st(s), on(p->opt.profile != 0) {
        if (on) P->n_timed = 0;
    }
    hipError_t begin(int32_t k, int64_t items) {
        if (!on) return hipSuccess;
        slot = P->n_timed++;
        if (P->timed.size() < P->n_timed) {
            qaoa_plan_s::Timed t{k, items, nullptr, nullptr};
            hipError_t e = hipEventCreate(&t.start);
            if (e == hipSuccess) e = hipEventCreate(&t.stop);
            if (e != hipSuccess) return e;
            P->timed.push_back(t);
        }
        P->timed[slot].k = k;
        P->timed[slot].items = items;
        return hipEventRecord(P->timed[slot].start, st);
    }
    hipError_t end() { return on ? hipEventRecord(P->timed[slot].stop, st) : hipSuccess; }
};

}  // namespace

// The gradient of a shared state of 14 qubits spills (about 1 KB a thread), and a point of its group
// occupies a compute unit for as long as several members' own states do: c times as long.  It is taken
// where the members would fill the chip c times as often.  Measured (us, energy and gradient, one
// shared state a point against filling the chip once, twice and three times with members): p = 2, up to
// 64, 128 and 256 points 43, 54 and 61 against 22, 36 and 50; p = 3 65, 82 and 95 against 33, 59 and
// 87; p = 5 100, 128 and 148 against 55, 104 and 153; p = 8 141, 188 and 212 against 88, 173 and
// 255; real weights, p = 2, 58, 70 and 77 against 35, 73 and 113.  13 qubits at p = 2: 20 against 18 and 28.
// Up to 12 qubits, and for energies alone, a shared state is never behind (12 qubits, p = 2, three members: 13
// and 14, 1 point; 101 and 275, 4096).
Shared shared_states(const qaoa_plan_s* P, bool grad, bool terms_read, int64_t n_points) {
    Shared s;
    s.Wg = P->d_W;
    if (P->wh_groups.empty() || terms_read) return s;
    auto fills = [&](int64_t n) { return (n * n_points + 255) / 256; };
    int sel = 0;
    for (const auto& cls : P->wh_groups) {
        int64_t c = 1;
        const int64_t states = cls.count * n_points;
        if (grad && cls.K == 14)
            c = P->hp.realw || (P->hp.p > 2 && states <= 64) ? 2 : P->hp.p > 3 || states <= (P->hp.p == 2 ? 64 : 128) ? 3 : 4;
        if (grad && cls.K == 13 && P->hp.p == 2) c = 2;
        if (fills(cls.members) < c * fills(cls.count)) continue;
        s.on[wh_class(cls.K) - 12] = true;
        if (cls.K > 12) sel |= 1 << (cls.K - 13);
    }
    s.Wg = P->d_Wg + static_cast<size_t>(sel) * P->hp.W.size();
    return s;
}

int Forms::runs(const qaoa_plan_s::Group& g, int64_t (&r)[2][2]) const {
    const bool s = sh.of(wh_class(g.K)), w = ((whole >> g.K) & 1u) != 0;
    const bool on[5] = {false, !s && w, !s, w, true};
    int n = 0;
    int64_t at = 0;
    for (int i = 0; i < 5; ++i) {
        const int64_t end = at + g.n_part[i];
        if (on[i] && end > at) {
            if (n > 0 && r[n - 1][1] == at) {
                r[n - 1][1] = end;
            } else {
                r[n][0] = at;
                r[n++][1] = end;
            }
        }
        at = end;
    }
    return n;
}

// Bands 1 and 2: a unit of a cone on its inner qubits takes a wave, however few amplitudes it has, where
// the kernel for whole cones holds many small cones in one; but a call's units share one launch, and
// whole cones take one per size.  So few units run on their inner qubits, many whole (in_small).
// Measured (ns an item where they fill the chip, inner and whole): p = 2, energies, 8, 9 and 10 qubits
// 1.5 and 0.4, 1.2 and 0.45, 1.0 and 0.7, 11 qubits 1.7 and 1.5; with the gradient 3.1 and 0.7, 2.7
// and 2.1, 2.2 and 4.2; p = 3, 8 to 11 qubits, gradient 7.5 and 1.2, 7.8 and 2.0, 8.9 and 4.4, 9.4
// and 11.6.
// Where they are the lesser part of the inner classes' workgroups, they hide behind the others.  Plans of
// up to four units have no idle waves: theirs of 10 qubits stay (a ring at p = 4, 8192 points: 78 us
// inner, 111 whole).
// Band 3: a wave takes a cone's rounds in series, where whole cones have a workgroup each, as many items as
// compute units.  Inner classes share a launch, as long as the cone of most rounds; whole cones take a
// launch a size, none more where cones of that size run whole anyway.  So the sizes of most rounds
// leave as long as that shortens the sum.  The estimates (us) are lines through measured latencies:
// p = 3, gradient, 12, 13 and 14 qubits in 2, 4 and 6 rounds 24, 42 and 60 inner, 21, 23 and 30 whole;
// energies 12, 18 and 25, and 11, 13 and 15.  Beyond 256 items the inner form is never behind (28
// cones of 14 qubits, 32 points: 64 and 112).
Forms choose_forms(const qaoa_plan_s* P, bool grad, bool terms_read, int64_t n_points) {
    Forms f;
    f.sh = shared_states(P, grad, terms_read, n_points);
    f.in = &P->in_groups;
    if (P->opt.tune != 0) {   // a layout is asked for, or chosen by timing
        f.whole = ~0u;   // (cones of tune = 1 that have both forms)
        return f;
    }
    if (P->in_bands.empty()) return f;
    const bool ten = !(grad && P->hp.p == 2) && !ten_stay(P);   // 10 qubits as well
    int64_t few = 0, blocks = 0;
    int32_t others = 0;   // rounds at most, outside band 3
    for (const auto& g : P->in_groups) {
        if (f.sh.of(g.wh) || g.tree) continue;
        others = std::max(others, g.rounds);
        few += g.small[ten ? 1 : 0];
        blocks += g.blocks[0];
    }
    if (few * n_points >= in_small(P->hp.p, grad) && 2 * few >= blocks) {
        f.whole = ten ? (1u << 11) - 1 : (1u << 10) - 1;
        f.in = &P->in_rest[ten ? 1 : 0];
        return f;
    }
    const size_t n = P->in_serial.size();
    if (n == 0) return f;
    const double layers = P->hp.p - 1, round = layers * (grad ? (P->hp.p == 2 ? 3.4 : 4.4) : 1.65);
    int64_t span[2][2];
    uint32_t runs = 0;   // sizes with a launch of whole cones
    for (const auto& g : P->lds_groups)
        if (f.runs(g, span) > 0) runs |= 1u << g.K;
    double moved = runs || !P->hbm_groups.empty() ? 0.0 : 3.5;   // phase rows
    double best = 0.0;
    uint32_t sizes = 0;
    for (size_t j = 0; j <= n; ++j) {   // the first j sizes whole
        int32_t left = others;
        for (const auto& b : P->in_bands)
            if (b.band == 3 && !f.sh.of(b.wh) && !((sizes >> b.K) & 1u)) left = std::max(left, b.rounds);
        const double t = (j ? moved : 0.0) + (left ? 6.0 + left * round : 0.0);
        if (j == 0 || t < best) {
            best = t;
            f.whole = sizes;
            f.in = j ? &P->in_rest[1 + j] : &P->in_groups;
        }
        if (j == n) break;
        const int K = P->in_serial[j];
        int64_t items = 0;
        for (const auto& b : P->in_bands)
            if (b.K == K && !f.sh.of(b.wh)) items += b.count * n_points;
        if (items > 256) break;
        if (items && !((runs >> K) & 1u))
            moved += grad ? 8.0 + layers * (K < 14 ? 0.5 * K + 1.0 : 10.5) : 5.5 + layers * (0.65 * K - 4.6);
        sizes |= 1u << K;
    }
    return f;
}

hipError_t launch_whole_group(const qaoa_plan_s* P, const qaoa_plan_s::WhGroup& grp, bool grad, int64_t n_points,
                              const double* gamma, const double* beta, int64_t gamma_P, double* zz, double* g,
                              hipStream_t st) {
    const HostPlan& hp = P->hp;
    WhArgs a{};
    a.groups = P->d_wh + grp.first;
    a.mem = P->d_whmem;
    a.cut = P->d_cut;
    a.obs = P->d_whobs;
    a.gamma = gamma;
    a.beta = beta;
    a.gamma_P = gamma_P;
    a.deltas = P->d_inst_delta;
    a.p = hp.p;
    a.cut_min = hp.cut_min;
    a.rowcap = grp.rowcap;
    a.realw = hp.realw ? 1 : 0;
    a.P = static_cast<int32_t>(n_points);
    a.M = static_cast<int32_t>(hp.cones.size());
    a.n_items = grp.count * n_points;
    a.zz = zz;
    a.g = g;
    if (!P->opt.one_cone_at_a_time) return launch_whole(grp.K, grad, a, st);
    for (int64_t n = a.n_items, it = 0; it < n; ++it) {
        a.item0 = it;
        a.n_items = it + 1;
        const hipError_t e = launch_whole(grp.K, grad, a, st);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

namespace {
InArgs inner_args(const qaoa_plan_s* P, const double* gamma, const double* beta, int64_t gamma_P, double* zz, double* g) {
    const HostPlan& hp = P->hp;
    InArgs a{};
    a.cones = P->d_in;
    a.cfg = P->d_incfg;
    a.grp = P->d_ingrp;
    a.leaf = P->d_leaf;
    a.wz = P->wz;
    a.tab = P->d_intab;
    a.gamma = gamma;
    a.beta = beta;
    a.gamma_P = gamma_P;
    a.deltas = P->d_inst_delta;
    a.p = hp.p;
    a.R = hp.cut_max - hp.cut_min + 1;
    a.cut_min = hp.cut_min;
    a.M = static_cast<int32_t>(hp.cones.size());
    a.zz = zz;
    a.g = g;
    return a;
}
D2Args depth2_args(const qaoa_plan_s* P, const double* gamma, const double* beta, int64_t gamma_P, double* zz, double* g) {
    D2Args a{};
    a.cones = P->d_tr;
    a.sides = P->d_sides;
    a.n_sides = P->n_sides;
    a.branch = P->d_branch;
    a.types = P->d_types;
    a.leaf = P->d_leaf2;
    a.n_types = P->n_types;
    a.gamma = gamma;
    a.beta = beta;
    a.gamma_P = gamma_P;
    a.deltas = P->d_inst_delta;
    a.M = static_cast<int32_t>(P->hp.cones.size());
    a.zz = zz;
    a.g = g;
    return a;
}

// The trees of a group.
hipError_t launch_tree_group(const qaoa_plan_s* P, const qaoa_plan_s::InGroup& grp, bool grad, int upw_log2,
                             int64_t n_points, const double* gamma, const double* beta, int64_t gamma_P, double* zz,
                             double* g, hipStream_t st) {
    D2Args a = depth2_args(P, gamma, beta, gamma_P, zz, g);
    if (P->opt.one_cone_at_a_time) {
        a.units = a.upw = a.blocks = a.n_seg = a.P = 1;
        for (int64_t i = 0; i < grp.count; ++i) {
            a.cones = P->d_tr + grp.first + i;
            a.inst0 = P->tr_inst[static_cast<size_t>(grp.first + i)];
            for (int64_t pt = 0; pt < n_points; ++pt) {
                a.point0 = static_cast<int32_t>(pt);
                const hipError_t e = launch_depth2(a, grad, st);
                if (e != hipSuccess) return e;
            }
        }
        return hipSuccess;
    }
    a.cones = P->d_tr + grp.first;
    a.units = static_cast<int32_t>(grp.count);
    a.upw = 1 << upw_log2;
    a.blocks = grp.blocks[upw_log2];
    a.n_seg = grp.n_seg;
    a.inst0 = P->tr_inst[static_cast<size_t>(grp.first)];
    a.seg = grp.n_seg > 1 ? P->d_inseg + grp.seg[upw_log2] : nullptr;
    // a grid holds fewer than 2^32 threads
    const int64_t slab = std::max<int64_t>(1, (static_cast<int64_t>(UINT32_MAX) / 256) / a.blocks);
    for (int64_t p0 = 0; p0 < n_points; p0 += slab) {
        a.point0 = static_cast<int32_t>(p0);
        a.P = static_cast<int32_t>(std::min(slab, n_points - p0));
        const hipError_t e = launch_depth2(a, grad, st);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}
}  // namespace

hipError_t launch_inner_group(const qaoa_plan_s* P, const qaoa_plan_s::InGroup& grp, bool grad, int upw_log2,
                              int64_t n_points, const double* gamma, const double* beta, int64_t gamma_P, double* zz,
                              double* g, double* part, size_t part_cap, hipStream_t st) {
    if (grp.tree) return launch_tree_group(P, grp, grad, upw_log2, n_points, gamma, beta, gamma_P, zz, g, st);
    const HostPlan& hp = P->hp;
    InArgs a = inner_args(P, gamma, beta, gamma_P, zz, g);
    a.cones = P->d_in + grp.first;
    a.signs = grp.signs ? 1 : 0;
    a.chunks = grp.chunks;
    a.part = part;
    const int64_t nv = grad ? 2 * hp.p + 1 : 1;
    auto run = [&](int64_t p0, int64_t np, int64_t cones) {
        a.point0 = static_cast<int32_t>(p0);
        a.P = static_cast<int32_t>(np);
        hipError_t e = launch_inner(grp.kin, grad, a, st);
        if (e == hipSuccess && grp.chunks > 1) e = launch_inner_sum(a, static_cast<int32_t>(cones), grad, st);
        return e;
    };
    if (P->opt.one_cone_at_a_time) {
        a.n_seg = 1;
        a.units = grp.chunks;
        a.upw = 1;
        a.blocks = (grp.chunks + 3) / 4;
        for (int64_t i = 0; i < grp.count; ++i) {
            a.cones = P->d_in + grp.first + i;
            a.inst0 = P->in_inst[static_cast<size_t>(grp.first + i)];
            for (int64_t pt = 0; pt < n_points; ++pt) {
                const hipError_t e = run(pt, 1, 1);
                if (e != hipSuccess) return e;
            }
        }
        return hipSuccess;
    }
    a.units = static_cast<int32_t>(grp.count * grp.chunks);
    a.upw = 1 << upw_log2;
    a.blocks = grp.blocks[upw_log2];
    a.n_seg = grp.n_seg;
    a.inst0 = P->in_inst[static_cast<size_t>(grp.first)];
    a.seg = grp.n_seg > 1 ? P->d_inseg + grp.seg[upw_log2] : nullptr;
    // points per launch: a grid holds fewer than 2^32 threads, and the partial sums their room
    auto slabs = [&](int64_t cones) {
        int64_t slab = std::max<int64_t>(1, (static_cast<int64_t>(UINT32_MAX) / 256) / a.blocks);
        if (grp.chunks > 1) slab = std::min(slab, static_cast<int64_t>(part_cap) / (a.units * nv));
        for (int64_t p0 = 0; p0 < n_points; p0 += slab) {
            const hipError_t e = run(p0, std::min(slab, n_points - p0), cones);
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    };
    const int64_t room = grp.chunks > 1 ? static_cast<int64_t>(part_cap) / (grp.chunks * nv) : grp.count;   // cones
    if (room >= grp.count) return slabs(grp.count);
    // the sums of a point's cones exceed a small memory budget: runs of cones of one instance (same bits)
    a.n_seg = 1;
    for (int64_t i = 0, j; i < grp.count; i = j) {
        a.inst0 = P->in_inst[static_cast<size_t>(grp.first + i)];
        for (j = i + 1; j < grp.count && j - i < room && P->in_inst[static_cast<size_t>(grp.first + j)] == a.inst0; ++j) {}
        a.cones = P->d_in + grp.first + i;
        a.units = static_cast<int32_t>((j - i) * grp.chunks);
        a.blocks = (a.units + 4 * a.upw - 1) / (4 * a.upw);
        const hipError_t e = slabs(j - i);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

qaoa_status kernel_times(qaoa_plan_s* P, int32_t cap, int32_t* k_out, int64_t* items_out, double* ms_out,
                         int32_t* n_out, std::string& msg) {
    if (!P->opt.profile || P->n_timed == 0) {
        msg = "plan was not built with profile = 1 or has not been evaluated";
        return QAOA_EINVAL;
    }
    for (size_t i = 0; i < P->n_timed && static_cast<int32_t>(i) < cap; ++i) {
        auto& t = P->timed[i];
        QCHECK(hipEventSynchronize(t.stop));
        float ms = 0.f;
        QCHECK(hipEventElapsedTime(&ms, t.start, t.stop));
        if (k_out) k_out[i] = t.k;
        if (items_out) items_out[i] = t.items;
        if (ms_out) ms_out[i] = ms;
    }
    if (n_out) *n_out = static_cast<int32_t>(P->n_timed);
    return QAOA_OK;
}

namespace {

// Device bytes of one (cone, point) item held as passes over device memory: its states (psi,
// lambda, or one state per checkpoint and lambda) and its partial sums.
size_t hbm_item_bytes(int k, int p, bool grad, bool ckpt) {
    const size_t state = (size_t{1} << (k - 1)) * sizeof(float2);
    const size_t sums = (size_t{1} << (k - 1 - HT)) * static_cast<size_t>(2 * p + 1) * sizeof(double);
    const size_t phi = p >= 2 ? (ckpt ? static_cast<size_t>(hbm_checkpoints(k, p)) : size_t{1}) * state : 0;
    return phi + (grad && p >= 2 ? state : 0) + sums;
}

// A memory budget that does not hold one item of a class is refused, also where the class runs
// without states of its own in device memory.
bool budget_refuses(const qaoa_plan_s* P, int k, bool grad, std::string& msg) {
    if (P->opt.mem_budget_bytes == 0) return false;
    const size_t budget = static_cast<size_t>(P->opt.mem_budget_bytes);
    const size_t need = hbm_item_bytes(k, P->hp.p, grad, grad && P->hp.p >= 2 && P->opt.checkpoint_mode == 1);
    if (budget >= need) return false;
    msg = "one " + std::to_string(k) + "-qubit item needs " + std::to_string(need) +
          " bytes, more than the memory budget of " + std::to_string(budget);
    return true;
}

// Orbit-weighted sums of the term rows zz, g (null: energies only) into E and dE.
qaoa_status finish_sums(qaoa_plan_s* P, int64_t n_points, double* zz, double* g, double* energy, double* dgamma,
                        double* dbeta, bool terms_read, const double* Wg, GroupTimer& tm, hipStream_t stream, std::string& msg) {
    const HostPlan& hp = P->hp;
    const int32_t p = hp.p, M = static_cast<int32_t>(hp.cones.size());
    const double* deltas = P->d_inst_delta;
    QCHECK(tm.begin(-2, n_points));
    if (terms_read) {
        // the caller reads the per-term gradient: gamma derivatives in radians (the combination
        // then scales by the unit once more, so it gets unit weights)
        bool unit = true;
        for (double d : hp.inst_delta) unit = unit && d == 1.0;
        if (!unit) {
            QCHECK(launch_scale_gamma_terms(g, n_points, p, M, P->d_inst_orbit, hp.n_inst, P->d_inst_delta, stream));
            deltas = P->d_ones;
        }
    }
    QCHECK(launch_combine(P->d_W, Wg, zz, g, M, p, P->d_inst_orbit, deltas, hp.n_inst, n_points, n_points, 0, energy,
                          dgamma, dbeta, stream));
    QCHECK(tm.end());
    return QAOA_OK;
}

// Values of partial sums that a call holds at most: 2^25, and where a memory budget is set, what it leaves
// beside one item of the largest class in device memory.  (A single cone's parts are always held:
// less than its state would take.)
size_t part_limit(const qaoa_plan_s* P) {
    constexpr size_t MOST = size_t{1} << 25;
    if (P->opt.mem_budget_bytes == 0) return MOST;
    const size_t budget = static_cast<size_t>(P->opt.mem_budget_bytes);
    size_t item = 0;
    for (const auto& grp : P->hbm_groups)
        item = std::max(item, hbm_item_bytes(grp.K, P->hp.p, true, P->hp.p >= 2 && P->opt.checkpoint_mode == 1));
    return std::min(MOST, (budget > item ? budget - item : 0) / sizeof(double));
}


// The launches of a depth-1 call.  One instance of few orbits: terms and weighted sums in one
// launch (2048 orbits are eight per thread of the point's workgroup; larger plans fill the chip
// better with a thread per term and a separate sum).
qaoa_status enqueue_depth1(qaoa_plan_s* P, int64_t n_points, const double* gamma, const double* beta, double* energy,
                           double* term_zz, double* dgamma, double* dbeta, double* term_grad, hipStream_t stream,
                           std::string& msg) {
    const HostPlan& hp = P->hp;
    const bool grad = dgamma != nullptr;
    const int32_t M = static_cast<int32_t>(hp.cones.size());
    if (P->max_k > P->opt.k_lds_max && budget_refuses(P, P->max_k, grad, msg)) return QAOA_ENOMEM;
    D1Args a{P->d_d1, P->d_d1w, M, gamma, beta, n_points, P->d_inst_delta, n_points, M, term_zz, term_grad, 1.0};
    if (hp.n_inst == 1 && M <= D1_POINT && !P->opt.profile && !P->opt.one_cone_at_a_time) {
        a.g_scale = hp.inst_delta[0];   // the caller's per-term gradient is in radians
        QCHECK(launch_depth1_point(a, P->d_W, energy, dgamma, dbeta, stream));
        return QAOA_OK;
    }
    qaoa_status st;
    if (!term_zz) {
        if ((st = grow(P->d_zz, P->cap_zz, static_cast<size_t>(n_points) * M, msg)) != QAOA_OK) return st;
        a.zz = P->d_zz;
    }
    if (grad && !term_grad) {
        if ((st = grow(P->d_g, P->cap_g, static_cast<size_t>(n_points) * 2 * M, msg)) != QAOA_OK) return st;
        a.g = P->d_g;
    }
    GroupTimer tm(P, stream);
    for (const auto& grp : P->d1_groups) {
        D1Args c = a;
        c.cones = P->d_d1 + grp.first;
        c.n_cones = grp.count;
        const int64_t items = grp.count * n_points;
        QCHECK(tm.begin(grp.K, items));
        if (P->opt.one_cone_at_a_time) {
            for (int64_t t = 0; t < items; ++t) QCHECK(launch_depth1_terms(c, t, t + 1, grad, stream));
        } else {
            QCHECK(launch_depth1_terms(c, 0, items, grad, stream));
        }
        QCHECK(tm.end());
    }
    return finish_sums(P, n_points, a.zz, a.g, energy, dgamma, dbeta, term_grad != nullptr, P->d_W, tm, stream, msg);
}

// A class's form in the tuner's keys: "tree", or inner qubits ("z": with leaves).
std::string inner_form(const qaoa_plan_s::InGroup& grp) {
    return grp.tree ? "tree" : std::to_string(grp.kin) + (grp.signs ? "z" : "");
}

// The next class of a shared launch.
InMix::Class& mix_class(const qaoa_plan_s* P, const qaoa_plan_s::InGroup& grp, InMix& mix) {
    InMix::Class& c = mix.c[mix.n++];
    c.kin = grp.kin;
    c.signs = grp.signs ? 1 : 0;
    c.cone0 = static_cast<int32_t>(grp.first);
    c.n_cones = static_cast<int32_t>(grp.count);
    c.units = static_cast<int32_t>(grp.count * grp.chunks);
    c.chunks = grp.chunks;
    c.block0 = mix.blocks;
    c.n_seg = grp.n_seg;
    c.inst0 = P->in_inst[static_cast<size_t>(grp.first)];
    c.seg = grp.n_seg > 1 ? P->d_inseg + grp.seg[0] : nullptr;
    mix.blocks += grp.blocks[0];
    return c;
}

// The cones on 11 to 14 inner qubits, as many of them per launch as the partial sums' room and the grid
// (fewer than 2^32 threads, 1024 per unit) hold, for as many points.  A cone's units and their order
// are its own: its sums do not depend on the split.
qaoa_status enqueue_wide(qaoa_plan_s* P, bool grad, int64_t n_points, const double* gamma, const double* beta, double* zz,
                         double* g, GroupTimer& tm, hipStream_t stream, std::string& msg) {
    const HostPlan& hp = P->hp;
    WdArgs a{};
    a.cones = P->d_wd;
    a.grp = P->d_wdgrp;
    a.leaf = P->d_wdleaf;
    a.wz = P->wz;
    a.cfg = P->d_wdcfg;
    a.tab = P->d_wdtab;
    a.gamma = gamma;
    a.beta = beta;
    a.gamma_P = n_points;
    a.deltas = P->d_inst_delta;
    a.p = hp.p;
    a.R = P->wd_rows;
    a.M = static_cast<int32_t>(hp.cones.size());
    a.part = P->d_part;
    a.zz = zz;
    a.g = g;
    const int64_t nv = grad ? 2 * hp.p + 1 : 1;
    const int64_t room = static_cast<int64_t>(P->cap_part) / nv;
    constexpr int64_t GRID = static_cast<int64_t>(UINT32_MAX) / 1024;
    const size_t n_cones = P->wd_units.size();
    for (size_t c0 = 0, c1; c0 < n_cones; c0 = c1) {
        const int64_t u0 = P->wd_units[c0].first;
        int64_t u1 = u0;
        for (c1 = c0; c1 < n_cones; ++c1) {
            const int64_t end = u1 + P->wd_units[c1].second;
            if (c1 > c0 && end - u0 > std::min(room, GRID)) break;
            u1 = end;
        }
        a.cone0 = static_cast<int32_t>(c0);
        a.sum_unit0 = static_cast<int32_t>(u0);
        a.all_units = static_cast<int32_t>(u1 - u0);
        // (a sum takes a workgroup of 256 threads per cone, which has one unit at least)
        const int64_t slab = std::max<int64_t>(1, std::min(room, GRID) / (u1 - u0));
        for (int64_t p0 = 0; p0 < n_points; p0 += slab) {
            const int32_t pc = static_cast<int32_t>(std::min(slab, n_points - p0));
            for (const auto& grp : P->wd_groups) {
                const int64_t first = std::max(grp.first, u0), last = std::min(grp.first + grp.count, u1);
                if (first >= last) continue;
                auto launch = [&](int64_t f, int64_t count, int64_t i0, int64_t np) {
                    a.units = P->d_wdunit + f;
                    a.unit0 = static_cast<int32_t>(f - u0);
                    a.n_units = static_cast<int32_t>(count);
                    a.point0 = static_cast<int32_t>(p0 + i0);
                    a.P = static_cast<int32_t>(np);
                    a.part = P->d_part + static_cast<size_t>(i0) * a.all_units * nv;
                    return launch_wide(grp.kin, grad, a, stream);
                };
                int64_t cones = 0;
                for (size_t c = c0; c < c1; ++c) cones += P->wd_units[c].first >= first && P->wd_units[c].first < last;
                QCHECK(tm.begin(grp.K, cones * pc));
                if (P->opt.one_cone_at_a_time) {
                    for (int64_t i = 0; i < pc; ++i)
                        for (size_t c = c0; c < c1; ++c)
                            if (P->wd_units[c].first >= first && P->wd_units[c].first < last)
                                QCHECK(launch(P->wd_units[c].first, P->wd_units[c].second, i, 1));
                } else {
                    QCHECK(launch(first, last - first, 0, pc));
                }
                QCHECK(tm.end());
            }
            a.point0 = static_cast<int32_t>(p0);
            a.P = pc;
            a.part = P->d_part;
            QCHECK(launch_wide_sum(a, static_cast<int32_t>(c1 - c0), grad, stream));
        }
    }
    return QAOA_OK;
}

// The launch sequence of one energy call.  With fixed_batches the HBM groups reuse the
// batch sizes of the previous call (and so allocate nothing): used while capturing.
qaoa_status enqueue(qaoa_plan_s* P, int64_t n_points, const double* gamma, const double* beta, double* energy,
                    double* term_zz, double* dgamma, double* dbeta, double* term_grad, hipStream_t stream,
                    bool fixed_batches,
                    std::string& msg) {
    qaoa_status st = ensure_device(P, msg);
    if (st != QAOA_OK) return st;
    if (depth1_closed(P))
        return enqueue_depth1(P, n_points, gamma, beta, energy, term_zz, dgamma, dbeta, term_grad, stream, msg);
    const HostPlan& hp = P->hp;
    const bool grad = (dgamma != nullptr);
    const int32_t p = hp.p;
    const int32_t M = static_cast<int32_t>(hp.cones.size());
    const int32_t R = hp.cut_max - hp.cut_min + 1;
    if (P->in_max_k > P->opt.k_lds_max && budget_refuses(P, P->in_max_k, grad, msg)) return QAOA_ENOMEM;
    if (P->d2_point) {
        D2Args a = depth2_args(P, gamma, beta, n_points, term_zz, grad ? term_grad : nullptr);
        a.units = M;
        a.P = static_cast<int32_t>(n_points);
        QCHECK(launch_depth2_point(a, P->d_W, energy, dgamma, dbeta, stream));
        return QAOA_OK;
    }
    const Forms forms = choose_forms(P, grad, grad && term_grad, n_points);
    // At p = 2 a point's workgroup waits for the slowest of its units, in 128 registers and 412 bytes of
    // scratch a thread; beyond what the chip holds at once their classes share a launch instead (a 12-node
    // graph of 15 orbits, energy and gradient, 512 points 55 -> 38 us; C_1000(1,2,3), 2048 points 365 ->
    // 288).  Deeper circuits sum in LDS either way (a path of 13 nodes, p = 4, 512 points: 67 here, 84).
    const bool crowd = p == 2 && P->in_point.n > 4 && P->in_point.n * n_points > 4096;
    if (!forms.whole && P->in_point.n && !crowd && !(P->in_parts.n && n_points * P->in_point.n <= IN_SPREAD)) {
        InArgs a = inner_args(P, gamma, beta, n_points, term_zz, grad ? term_grad : nullptr);
        InPoint q = P->in_point;
        q.W = P->d_W;
        q.energy = energy;
        q.dgamma = dgamma;
        q.dbeta = dbeta;
        QCHECK(launch_inner_point(a, depth2_args(P, gamma, beta, n_points, nullptr, nullptr), q, grad, n_points, stream));
        return QAOA_OK;
    }
    if (!forms.whole && P->in_parts.n && n_points <= IN_MIX) {
        // few cones: their classes in one launch, then all sums
        const int64_t nvals = grad ? 2 * p + 1 : 1;
        InMix mix{};
        InPointSum q = P->in_parts;
        int64_t parts = 0, units = 0, cone = 0;
        mix.all = 1;
        for (const auto& grp : P->in_groups) {
            units = std::max(units, grp.count * grp.chunks * n_points);
            mix_class(P, grp, mix).part0 = parts;
            for (int64_t c = 0; c < grp.count; ++c) q.c[cone++].part0 = parts;
            parts += grp.count * grp.chunks * n_points * nvals;
        }
        if (units <= IN_MIX && parts <= static_cast<int64_t>(part_limit(P))) {
            if ((st = grow(P->d_part, P->cap_part, static_cast<size_t>(parts), msg)) != QAOA_OK) return st;
            InArgs a = inner_args(P, gamma, beta, n_points, term_zz, grad ? term_grad : nullptr);
            a.part = P->d_part;
            a.P = static_cast<int32_t>(n_points);
            QCHECK(launch_inner_mix(a, mix, grad, stream));
            q.W = P->d_W;
            q.energy = energy;
            q.dgamma = dgamma;
            q.dbeta = dbeta;
            QCHECK(launch_inner_point_sum(a, q, grad, stream));
            return QAOA_OK;
        }
    }
    const size_t npl = static_cast<size_t>(hp.n_inst) * n_points * p;   // (instance, point, layer) rows
    const Shared& sh = forms.sh;
    int64_t span[2][2];   // a size's runs of cones on the kernel for whole cones
    // phase and mixer tables, for the kernels that read them
    bool tables = !P->hbm_groups.empty();
    for (const auto& grp : P->lds_groups) tables = tables || forms.runs(grp, span) > 0;
    if (tables) {
        if ((st = grow(P->d_phase, P->cap_phase, npl * R, msg)) != QAOA_OK) return st;
        if ((st = grow(P->d_mix, P->cap_mix, npl, msg)) != QAOA_OK) return st;
    }
    double* zz = term_zz;
    if (!zz) {
        if ((st = grow(P->d_zz, P->cap_zz, static_cast<size_t>(n_points) * M, msg)) != QAOA_OK) return st;
        zz = P->d_zz;
    }
    double* g = nullptr;
    if (grad && term_grad) {
        g = term_grad;
    } else if (grad) {
        if ((st = grow(P->d_g, P->cap_g, static_cast<size_t>(n_points) * 2 * p * M, msg)) != QAOA_OK) return st;
        g = P->d_g;
    }
    // partial sums of cones in several units: a cone's at least
    size_t part_need = 0;
    const size_t part_most = part_limit(P);
    const size_t nv = grad ? 2 * static_cast<size_t>(p) + 1 : 1;
    const std::vector<qaoa_plan_s::InGroup>& classes = *forms.in;
    for (const auto& grp : classes)
        if (grp.chunks > 1) {
            const size_t one = static_cast<size_t>(grp.chunks) * nv;
            part_need = std::max(part_need, std::max(one, std::min(one * grp.count * n_points, part_most)));
        }
    // classes that share a launch, with room for the sums of all their parts
    InMix mix{};
    std::vector<char> mixed(classes.size(), 0);
    if (!P->opt.profile && P->opt.tune == 0 && !P->opt.one_cone_at_a_time && n_points <= IN_MIX) {
        int64_t parts = 0;
        for (size_t i = 0; i < classes.size() && mix.n < IN_CLASSES; ++i) {
            const auto& grp = classes[i];
            const int64_t units = grp.count * grp.chunks;
            if (grp.tree || sh.of(grp.wh) || units * n_points > IN_MIX ||
                (grp.chunks > 1 && parts + units * n_points * static_cast<int64_t>(nv) > static_cast<int64_t>(part_most)))
                continue;
            InMix::Class& c = mix_class(P, grp, mix);
            c.part0 = parts;
            c.item0 = mix.items;
            if (grp.chunks > 1) {
                parts += units * n_points * static_cast<int64_t>(nv);
                mix.items += grp.count * n_points * static_cast<int64_t>(nv);
            }
            mixed[i] = 1;
        }
        if (mix.n < 2) {
            mix = InMix{};
            std::fill(mixed.begin(), mixed.end(), char{0});
        } else {
            part_need = std::max(part_need, static_cast<size_t>(parts));
        }
    }
    if (!P->wd_units.empty()) {   // a cone's at least
        const size_t all = static_cast<size_t>(P->wd_all_units) * nv * static_cast<size_t>(n_points);
        part_need = std::max({part_need, static_cast<size_t>(P->wd_most_units) * nv, std::min(all, part_most)});
    }
    if (part_need && (st = grow(P->d_part, P->cap_part, part_need, msg)) != QAOA_OK) return st;
    GroupTimer tm(P, stream);
    if (tables) {
        QCHECK(tm.begin(-1, static_cast<int64_t>(npl)));
        QCHECK(launch_tables(gamma, beta, static_cast<int64_t>(npl), R, hp.cut_min, P->d_inst_delta,
                             static_cast<int64_t>(n_points) * p, P->d_phase, P->d_mix, stream));
        QCHECK(tm.end());
    }
    EvalArgs ea{static_cast<int32_t>(n_points), p, M, R, P->d_phase, P->d_mix, gamma,
                static_cast<int32_t>(n_points), hp.realw ? 1 : 0, zz, g};
    const std::string arch = P->opt.tune == 1 ? device_arch(P->device) : std::string();
    // units per wave: the workgroup's set-up (phase rows) is shared by more units once the waves
    // fill the chip several times over
    auto inner_upw = [&](const qaoa_plan_s::InGroup& grp, int64_t points) {
        const int64_t units = grp.count * grp.chunks * points / (grp.tree ? 64 : 1);
        int j = 0;
        while (j < 3 && (units >> (j + 1)) >= (int64_t{1} << (grp.tree ? 13 : 15))) ++j;
        return j;
    };
    auto run_inner = [&](const qaoa_plan_s::InGroup& grp, int j, int64_t points) {   // the call's first points
        return launch_inner_group(P, grp, grad, j, points, gamma, beta, n_points, zz, g, P->d_part, P->cap_part, stream);
    };
    if (mix.n) {
        InArgs a = inner_args(P, gamma, beta, n_points, zz, g);
        a.part = P->d_part;
        a.P = static_cast<int32_t>(n_points);
        QCHECK(launch_inner_mix(a, mix, grad, stream));
        QCHECK(launch_inner_mix_sum(a, mix, grad, stream));
    }
    for (const auto& grp : classes) {
        if (sh.of(grp.wh) || mixed[static_cast<size_t>(&grp - classes.data())]) continue;
        if (P->opt.tune == 1 && grp.K <= P->opt.k_lds_max) continue;   // with the other cones of its size, below
        int j = inner_upw(grp, n_points);
        if (P->opt.tune == 1) {
            const TuneKey key{arch, 2, grp.K, p, grad ? 1 : 0, 0, inner_form(grp)};
            int upw = 1 << j;
            if (!tune_lookup(key, upw) && !fixed_batches)
                QCHECK(tune_pick(key, {1, 2, 4, 8}, grp.count * n_points, stream,
                                 [&](int v) { return run_inner(grp, __builtin_ctz(static_cast<unsigned>(v)), n_points); }, upw));
            j = __builtin_ctz(static_cast<unsigned>(std::min(upw, 8)));
        }
        QCHECK(tm.begin(grp.K, grp.count * n_points));
        QCHECK(run_inner(grp, j, n_points));
        QCHECK(tm.end());
    }
    if (!P->wd_units.empty()) {
        st = enqueue_wide(P, grad, n_points, gamma, beta, zz, g, tm, stream, msg);
        if (st != QAOA_OK) return st;
    }
    for (const auto& grp : P->wh_groups) {
        if (!sh.of(wh_class(grp.K))) continue;
        QCHECK(tm.begin(grp.K, grp.members * n_points));
        QCHECK(launch_whole_group(P, grp, grad, n_points, gamma, beta, n_points, zz, g, stream));
        QCHECK(tm.end());
    }
    // the first n items of one cone size in layout v; the default (0) takes the cones with a shell, which
    // come first, on their inner qubits (tune = 1 plans hold them in both forms): of n items all of these
    // cones at the first points, where the other layouts take the first cones at all points
    auto run_size = [&](const qaoa_plan_s::Group& grp, int v, int64_t n) {
        int64_t done = 0;
        if (v == 0 && grp.n_in > 0) {
            const int64_t points = std::min(n_points, n / grp.n_in);
            for (const auto& ig : P->in_groups)
                if (ig.K == grp.K) {
                    const hipError_t e = run_inner(ig, inner_upw(ig, points), points);
                    if (e != hipSuccess) return e;
                }
            done = grp.n_in * n_points;
        }
        if (done >= n) return hipSuccess;
        return launch_fused(grp.K, grad, v, P->d_cones + grp.first, done, n, P->d_cut, grp.rowcap, ea, stream);
    };
    for (const auto& grp : P->lds_groups) {
        const ConeDev* cones = P->d_cones + grp.first;
        const int64_t items = grp.count * n_points;
        const int n_runs = forms.runs(grp, span);
        if (n_runs == 0) continue;
        int variant = P->opt.tune >= 2 ? P->opt.tune - 2 : 0;   // tune 2, 3, 4: a fixed layout variant
        if (P->opt.tune == 1 && !P->opt.one_cone_at_a_time) {
            std::string form;   // of the size's cones: those on their inner qubits, "+" others
            for (const auto& ig : P->in_groups)
                if (ig.K == grp.K) form += (form.empty() ? "" : ",") + inner_form(ig);
            if (!form.empty() && grp.n_in < grp.count) form += "+";
            const TuneKey key{arch, 0, grp.K, p, grad ? 1 : 0, hp.realw ? 1 : 0, form};
            if (!tune_lookup(key, variant)) {
                const std::vector<int> cand = fused_variants(grp.K, grad);
                if (cand.size() <= 1 || fixed_batches) {
                    variant = 0;
                } else {
                    // timed on up to 2^16 items of this call (their results are written again below)
                    int64_t ns = std::min<int64_t>(items, int64_t{1} << 16);
                    if (grp.n_in * n_points > ns) ns = std::max<int64_t>(1, ns / grp.n_in) * grp.n_in;   // whole points
                    QCHECK(tune_pick(key, cand, ns, stream, [&](int v) {
                        return run_size(grp, v, ns);
                    }, variant));
                }
            }
        }
        int64_t n_run = 0;
        for (int r = 0; r < n_runs; ++r) n_run += span[r][1] - span[r][0];
        QCHECK(tm.begin(grp.K, n_run * n_points));
        if (P->opt.one_cone_at_a_time) {
            for (int r = 0; r < n_runs; ++r)
                for (int64_t it = span[r][0] * n_points; it < span[r][1] * n_points; ++it)
                    QCHECK(launch_fused(grp.K, grad, 0, cones, it, it + 1, P->d_cut, grp.rowcap, ea, stream));
        } else if (P->opt.tune == 1) {
            QCHECK(run_size(grp, variant, items));
        } else {
            for (int r = 0; r < n_runs; ++r)
                QCHECK(launch_fused(grp.K, grad, variant, cones, span[r][0] * n_points, span[r][1] * n_points, P->d_cut,
                                    grp.rowcap, ea, stream));
        }
        QCHECK(tm.end());
    }
    // ---- HBM-resident cones: batches of items through the pass program
    if (!fixed_batches) {
        P->hbm_batch.assign(P->hbm_groups.size(), 0);
        P->hbm_ckpt.assign(P->hbm_groups.size(), 0);
        std::fill(std::begin(P->pass_launches), std::end(P->pass_launches), int64_t{0});
        P->checkpointed_classes = 0;
        P->checkpointed_k_mask = 0;
    }
    for (size_t gi = 0; gi < P->hbm_groups.size(); ++gi) {
        const auto& grp = P->hbm_groups[gi];
        const int k = grp.K, kh = k - 1;      // stored qubits: the half with qubit k-1 = 0
        const int64_t items = grp.count * n_points;
        const int64_t tiles = int64_t{1} << (kh - HT);
        const int nvals = grad ? 2 * p + 1 : 1;     // values reduced per item
        const int stride = 2 * p + 1;                // values stored per (item, tile)
        const bool need_phi = p >= 2;
        const bool need_lam = grad && p >= 2;
        // checkpoints: every forward pass but the final one keeps its output (nck states)
        const int nck = hbm_checkpoints(k, p);
        const size_t per_unc = hbm_item_bytes(k, p, grad, false);
        const size_t per_ck = hbm_item_bytes(k, p, grad, true);
        size_t budget = static_cast<size_t>(P->opt.mem_budget_bytes);
        if (!fixed_batches && budget == 0) {
            size_t fr = 0, tot = 0;
            QCHECK(hipMemGetInfo(&fr, &tot));
            const size_t held = P->cap_phi * sizeof(float2) + P->cap_lam * sizeof(float2) + P->cap_gpart * sizeof(double);
            budget = static_cast<size_t>(0.85 * static_cast<double>(fr + held));
        } else if (!fixed_batches) {   // less the partial sums of other cones, down to one item (part_limit)
            const size_t item = P->opt.checkpoint_mode == 1 ? per_ck : per_unc, parts = P->cap_part * sizeof(double);
            if (budget > item) budget = budget - item > parts ? budget - parts : item;
        }
        // tiles (group 0: tile pairs) per workgroup: up to 8 while the class keeps >= 4096
        // workgroups (16 per CU); fixed per class, so an item's sums run in the same order
        // whatever the batching
        int tpw = 1;
        while (tpw < 8 && 2 * tpw <= tiles / 2 && items * tiles / (2 * tpw) >= 4096) tpw *= 2;
        const TuneKey tkey{arch, 1, k, p, grad ? 1 : 0, 0, ""};
        bool tune_tpw = false;
        if (P->opt.tune == 1) {
            int c = 0;
            if (tune_lookup(tkey, c)) tpw = c;
            else tune_tpw = !fixed_batches;
        }
        // items per batch: within the budget, the grid (a pass launches up to tiles * B
        // workgroups of <= 512 threads: below 2^31 work-items) and no more than needed for
        // 2^17 workgroups (512 per CU) per pass: larger batches hold more memory and gain little
        auto batch_of = [&](size_t per_item) {
            int64_t B = std::min<int64_t>(static_cast<int64_t>(budget / per_item), items);
            B = std::min<int64_t>(B, std::max<int64_t>(1, (int64_t{1} << 22) / tiles));
            return std::min<int64_t>(B, std::max<int64_t>(1, ((int64_t{1} << 17) * tpw + tiles - 1) / tiles));
        };
        bool ckpt = false;
        if (grad && p >= 2) {
            if (fixed_batches) ckpt = P->hbm_ckpt[gi] != 0;
            else if (P->opt.checkpoint_mode == 1) ckpt = true;
            // auto: store the forward states where the budget holds them without shrinking the
            // batch, or with a batch that still gives every pass 2^15 workgroups (128 per CU)
            else if (P->opt.checkpoint_mode == 2)
                ckpt = budget >= per_ck && (batch_of(per_ck) >= batch_of(per_unc) ||
                                            batch_of(per_ck) * tiles / (2 * tpw) >= (int64_t{1} << 15));
        }
        const size_t per_item = ckpt ? per_ck : per_unc;
        const int nphi = ckpt ? nck : 1;
        int64_t B;
        if (fixed_batches) {
            B = P->hbm_batch[gi];
        } else {
            if (budget < per_item) {
                msg = "one " + std::to_string(k) + "-qubit item needs " + std::to_string(per_item) +
                      " bytes, more than the memory budget of " + std::to_string(budget);
                return QAOA_ENOMEM;
            }
            B = batch_of(per_item);
        }
        // free memory can be fragmented or held by other allocators: on a failed allocation
        // the batch is halved until one item does not fit either
        for (;;) {
            st = QAOA_OK;
            if (need_phi) st = grow(P->d_phi, P->cap_phi, (static_cast<size_t>(B) * nphi) << kh, msg);
            if (st == QAOA_OK && need_lam) st = grow(P->d_lam, P->cap_lam, static_cast<size_t>(B) << kh, msg);
            if (st == QAOA_OK) st = grow(P->d_gpart, P->cap_gpart, static_cast<size_t>(B) * tiles * stride, msg);
            if (st != QAOA_ENOMEM || B == 1) break;
            for (float2** b : {&P->d_phi, &P->d_lam}) {
                hipFree(*b);
                *b = nullptr;
            }
            P->cap_phi = P->cap_lam = 0;
            B /= 2;
        }
        if (st != QAOA_OK) return st;
        P->hbm_batch[gi] = B;
        P->hbm_ckpt[gi] = ckpt ? 1 : 0;
        if (!fixed_batches && ckpt) {
            P->checkpointed_classes += 1;
            P->checkpointed_k_mask |= 1u << k;
        }
        const std::vector<PassSpec> prog = hbm_program(k, p, grad, ckpt);
        auto slot = [&](int j) { return P->d_phi + ((static_cast<size_t>(std::max(j, 0)) * B) << kh); };
        QCHECK(tm.begin(k, items));
        auto pass_args = [&](const PassSpec& ps, int64_t i0, int64_t nb) {
            PassArgs pa{};
            pa.cones = P->d_hcones + grp.first;
            pa.e_a = P->d_ea;
            pa.e_b = P->d_eb;
            pa.e_w = P->d_ew;
            pa.e_wd = P->d_ewd;
            pa.tt = P->d_tt;
            pa.phi_in = slot(ps.ck_in);
            pa.phi = ps.kind >= RV_GEN_MIX ? slot(ps.ck_in) : slot(ps.ck_out);
            pa.store_phi = ps.store_phi;
            pa.lam = P->d_lam;
            pa.gpart = P->d_gpart;
            pa.item0 = i0;
            pa.n_batch = static_cast<int32_t>(nb);
            pa.k = k;
            pa.kh = kh;
            pa.group = ps.group;
            pa.la = ps.la;
            pa.lb = ps.lb;
            pa.m0a = ps.m0a;
            pa.m0b = ps.m0b;
            pa.rowcap = grp.rowcap;
            pa.fix_layer = ps.fix_layer;
            pa.fix_pow = ps.fix_pow;
            pa.tpw = tpw;
            pa.ea = ea;
            return pa;
        };
        if (tune_tpw) {
            // tiles per workgroup: the class's first pass on its first batch (a generating
            // pass: it reads no state, and the partial sums it adds are cleared below)
            std::vector<int> cand;
            const int64_t units = tiles / 2;   // tile pairs of group 0 (the fewest units)
            for (int c = 1; c <= 8; c *= 2)
                if (c <= units && units % c == 0) cand.push_back(c);
            const int64_t nb = std::min<int64_t>(B, items);
            QCHECK(tune_pick(tkey, cand, nb, stream, [&](int c) {
                PassArgs pa = pass_args(prog[0], 0, nb);
                pa.tpw = c;
                return launch_pass(prog[0].kind, pa, stream);
            }, tpw));
        }
        for (int64_t i0 = 0; i0 < items; i0 += B) {
            const int64_t nb = std::min<int64_t>(B, items - i0);
            QCHECK(launch_fill_zero(P->d_gpart, nb * tiles * stride, stream));
            for (const PassSpec& ps : prog) {
                const PassArgs pa = pass_args(ps, i0, nb);
                QCHECK(launch_pass(ps.kind, pa, stream));
                if (!fixed_batches) P->pass_launches[ps.kind] += 1;
            }
            QCHECK(launch_tile_reduce(P->d_hcones + grp.first, P->d_gpart, i0, nb, tiles, stride, nvals, ea, stream));
        }
        QCHECK(tm.end());
    }
    return finish_sums(P, n_points, zz, g, energy, dgamma, dbeta, grad && term_grad, sh.Wg, tm, stream, msg);
}

void drop_graph(qaoa_plan_s* P) {
    if (P->gexec) hipGraphExecDestroy(P->gexec);
    P->gexec = nullptr;
    P->gkey = qaoa_plan_s::GraphKey{};
}

}  // namespace

namespace {
qaoa_status run_energy_throwing(qaoa_plan_s* P, int64_t n_points, const double* gamma, const double* beta,
                                double* energy, double* term_zz, double* dgamma, double* dbeta, double* term_grad,
                                hipStream_t stream, std::string& msg) {
    if (!P->opt.graph)
        return enqueue(P, n_points, gamma, beta, energy, term_zz, dgamma, dbeta, term_grad, stream, false, msg);
    qaoa_plan_s::GraphKey key;
    key.n_points = n_points;
    key.grad = dgamma != nullptr;
    const void* ptrs[7] = {gamma, beta, energy, term_zz, dgamma, dbeta, term_grad};
    for (int i = 0; i < 7; ++i) key.ptr[i] = ptrs[i];
    if (P->gexec && key == P->gkey) {
        QCHECK(hipGraphLaunch(P->gexec, stream));
        ++P->graph_replays;
        return QAOA_OK;
    }
    // a new key: run eagerly (allocating what the call needs), then capture the same launch
    // sequence on the plan's own stream; the graph is replayed from the next call on
    drop_graph(P);
    qaoa_status st = enqueue(P, n_points, gamma, beta, energy, term_zz, dgamma, dbeta, term_grad, stream, false, msg);
    if (st != QAOA_OK) return st;
    if (!P->cap_stream) QCHECK(hipStreamCreateWithFlags(&P->cap_stream, hipStreamNonBlocking));
    QCHECK(hipStreamBeginCapture(P->cap_stream, hipStreamCaptureModeThreadLocal));
    st = enqueue(P, n_points, gamma, beta, energy, term_zz, dgamma, dbeta, term_grad, P->cap_stream, true, msg);
    hipGraph_t graph = nullptr;
    const hipError_t ec = hipStreamEndCapture(P->cap_stream, &graph);
    if (st == QAOA_OK && ec != hipSuccess) {
        msg = std::string("hipStreamEndCapture: ") + hipGetErrorString(ec);
        st = QAOA_EHIP;
    }
    if (st == QAOA_OK) {
        const hipError_t ei = hipGraphInstantiate(&P->gexec, graph, nullptr, nullptr, 0);
        if (ei != hipSuccess) {
            msg = std::string("hipGraphInstantiate: ") + hipGetErrorString(ei);
            P->gexec = nullptr;
            st = QAOA_EHIP;
        }
    }
    if (graph) hipGraphDestroy(graph);
    if (st == QAOA_OK) P->gkey = key;
    return st;
}
}  // namespace

// The upload of a first call plans on the host: its allocation failures end here, not at the
// C boundary.
qaoa_status run_energy(qaoa_plan_s* P, int64_t n_points, const double* gamma, const double* beta, double* energy,
                       double* term_zz, double* dgamma, double* dbeta, double* term_grad, hipStream_t stream,
                       std::string& msg) {
    try {
        return run_energy_throwing(P, n_points, gamma, beta, energy, term_zz, dgamma, dbeta, term_grad, stream, msg);
    } catch (const std::bad_alloc&) {
        msg = "host allocation failed";
        return QAOA_ENOMEM;
    }
}

std::string tuning_report() {
    std::lock_guard<std::mutex> lk(g_tune_mu);
    std::string out;
    char line[256];
    for (const auto& kv : g_tune) {
        const TuneKey& key = kv.first;
        const TuneRec& r = kv.second;
        std::snprintf(line, sizeof(line), "%s %s k=%d p=%d grad=%d realw=%d", key.arch.c_str(),
                      key.what == 0 ? "workgroup-variant" : "passes-tiles-per-workgroup", key.k, key.p, key.grad, key.realw);
        out += line;
        if (!key.form.empty()) out += " form=" + key.form;
        std::snprintf(line, sizeof(line), " items=%lld choice=%d ms:", static_cast<long long>(r.items), r.choice);
        out += line;
        for (const auto& cm : r.ms) {
            std::snprintf(line, sizeof(line), " %d=%.4f", cm.first, cm.second);
            out += line;
        }
        out += "\n";
    }
    return out;
}

void release_device(qaoa_plan_s* P) {
    drop_graph(P);
    if (P->cap_stream) {
        hipStreamDestroy(P->cap_stream);
        P->cap_stream = nullptr;
    }
    for (auto& t : P->timed) {
        hipEventDestroy(t.start);
        hipEventDestroy(t.stop);
    }
    P->timed.clear();
    if (!P->dev_ready && !P->d_arena && !P->d_phase) return;
    hipDeviceSynchronize();
    hipFree(P->d_arena);
    hipFree(P->d_phase);
    hipFree(P->d_mix);
    hipFree(P->d_zz);
    hipFree(P->d_g);
    hipFree(P->d_phi);
    hipFree(P->d_lam);
    hipFree(P->d_gpart);
    hipFree(P->d_part);
    P->d_arena = nullptr;
    P->d_cones = nullptr;
    P->d_d1 = nullptr;
    P->d_d1w = nullptr;
    P->d_cut = nullptr;
    P->d_W = nullptr;
    P->d_hcones = nullptr;
    P->d_ea = P->d_eb = P->d_ew = nullptr;
    P->d_ewd = nullptr;
    P->d_tt = nullptr;
    P->d_inst_orbit = nullptr;
    P->d_inst_delta = nullptr;
    P->d_ones = nullptr;
    P->d_phi = P->d_lam = nullptr;
    P->d_gpart = nullptr;
    P->d_part = nullptr;
    P->cap_part = 0;
    P->d_in = nullptr;
    P->d_ingrp = nullptr;
    P->d_leaf = P->d_wdleaf = nullptr;
    P->d_tr = nullptr;
    P->d_sides = nullptr;
    P->d_branch = nullptr;
    P->d_types = nullptr;
    P->d_leaf2 = nullptr;
    P->d_intab = nullptr;
    P->d_wd = nullptr;
    P->d_wdunit = nullptr;
    P->d_wdgrp = nullptr;
    P->d_wdcfg = nullptr;
    P->d_wdtab = nullptr;
    P->d_incfg = nullptr;
    P->d_inseg = nullptr;
    P->cap_phi = P->cap_lam = P->cap_gpart = 0;
    P->d_phase = nullptr;
    P->d_mix = nullptr;
    P->d_zz = nullptr;
    P->d_g = nullptr;
    P->cap_phase = P->cap_mix = P->cap_zz = P->cap_g = 0;
    P->dev_ready = false;
}

}  // namespace qaoa
