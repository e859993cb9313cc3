// Host planning of cones evaluated on their inner qubits (inner_plan.hpp).
#include "inner_plan.hpp"

#include "pool.hpp"

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <new>
#include <thread>

namespace qaoa {

bool ShellPlanner::Shape::same(const Shape& o) const {
    return kin == o.kin && grp.size() == o.grp.size() && std::memcmp(level, o.level, sizeof(level)) == 0 &&
           std::memcmp(w, o.w, sizeof(w)) == 0 && std::memcmp(leaf, o.leaf, sizeof(leaf)) == 0 &&
           (grp.empty() || std::memcmp(grp.data(), o.grp.data(), grp.size() * sizeof(ShellGroup)) == 0);
}

namespace {
uint64_t mix64(uint64_t x) {
    x *= 0x9E3779B97F4A7C15ull;
    x ^= x >> 29;
    return x * 0xBF58476D1CE4E5B9ull;
}
}  // namespace

// The configurations of a shell up to the symmetries that keep a term: automorphisms of the inner
// qubits with their couplings, distance classes, leaves and shell groups (which may swap u and v),
// and the flip of all qubits (which keeps a term for any signs).  Configurations are tuples of
// digits, one per group (how many of its qubits are 1) and one per qubit with leaves (its sign).
// Twins (qubits of one class that a transposition swaps, each with digits of its own) are kept
// sorted by their digits; the remaining automorphisms, found by backtracking up to orders of
// twins, and the flip map sorted tuples to each other, and the smallest image of each orbit is
// listed with the weight of all its members.  What is listed depends on the shape alone, so a
// term is the same in every plan.  Where a wave holds them all at once, only the flip is used (the
// search for symmetries takes 4 us of host time a shape).  Up to 1024 configurations are always listed (under 0.3 ms of
// host time).  Beyond, up to 16384: at most 10 inner qubits, where a configuration costs a wave
// under 1 us, where at least 16 symmetries shorten the list enough to pay for it; more, where
// each occupies a compute unit for 37 us, with any symmetry at all.  No list: cfg stays empty.
void ShellPlanner::Shape::enumerate() {
    const uint32_t nh = (nc + 1) / 2, n_sign = 1u << __builtin_popcount(zmask);
    if (kin <= 10 && nh <= 64u && nh * n_sign <= (64u >> std::max(0, kin - 4))) {
        for (const ShellGroup& q : grp)
            if (q.m > 29) return;
        for (uint32_t d = 0; d < nh; ++d) {
            ShellCfg e{};
            e.w = (nc & 1u) && d == nh - 1 ? 1.0 : 2.0;
            uint32_t rem = d;
            for (const ShellGroup& G : grp) {
                const int t = static_cast<int>(rem % static_cast<uint32_t>(G.m + 1));
                rem /= static_cast<uint32_t>(G.m + 1);
                e.c0 += t * G.wsum;
                for (int i = 0; i < SH_H; ++i) e.h[i] = static_cast<int16_t>(e.h[i] + (G.m - 2 * t) * G.h[i]);
                for (int i = 0; i < t; ++i) e.w = e.w * (G.m - i) / (i + 1);
            }
            for (uint32_t s = 0; s < n_sign; ++s) {
                e.z = 0;
                uint32_t r = s;
                for (uint32_t z = zmask; z; z &= z - 1, r >>= 1) e.z |= (r & 1u) << __builtin_ctz(z);
                cfg.push_back(e);
            }
        }
        return;
    }
    std::vector<ShellGroup> grp = this->grp;   // and one of a single qubit for each sign
    const int n_real = static_cast<int>(grp.size());
    for (uint32_t z = zmask; z; z &= z - 1) {
        const int a = __builtin_ctz(z);
        int like = 0;
        while (std::memcmp(&leaf[like], &leaf[a], sizeof(leaf[a])) != 0) ++like;
        ShellGroup g;
        g.m = 1;
        g.wsum = INT32_MIN + like;             // its leaves; no sum of couplings
        g.h[a - 2] = 1;
        grp.push_back(g);
    }
    const int ng = static_cast<int>(grp.size());
    const uint64_t n_tuple = static_cast<uint64_t>(nc) << (ng - n_real);
    std::vector<ShellCfg>& out = cfg;
    if (n_tuple < 2 || n_tuple > 16384 || ng > 16) return;
    for (const ShellGroup& q : grp)
        if (q.m > 15) return;
    // groups private to one inner qubit, and twin classes
    std::vector<int> owner(ng, -1);
    std::vector<std::vector<int>> priv(kin);
    for (int q = 0; q < ng; ++q) {
        int n = 0, at = -1;
        for (int i = 0; i < SH_H; ++i)
            if (grp[q].h[i]) { ++n; at = i + 2; }
        if (n == 1) {
            owner[q] = at;
            priv[at].push_back(q);
        }
    }
    auto swapped = [](int x, int a, int b) { return x == a ? b : x == b ? a : x; };
    auto find_group = [&](const ShellGroup& want) {
        for (int q = 0; q < ng; ++q)
            if (std::memcmp(&grp[q], &want, sizeof(ShellGroup)) == 0) return q;
        return -1;
    };
    // image of group q under the qubit map sigma, or -1
    auto image = [&](int q, const int* sigma) {
        ShellGroup x = grp[q];
        for (int i = 0; i < SH_H; ++i) x.h[i] = 0;
        for (int i = 0; i < SH_H; ++i)
            if (grp[q].h[i]) x.h[sigma[i + 2] - 2] = grp[q].h[i];
        return find_group(x);
    };
    std::vector<int> cls(kin, -1);
    std::vector<std::vector<int>> classes;
    for (int a = 2; a < kin; ++a) {
        if (cls[a] >= 0) continue;
        std::vector<int> c{a};
        for (int b = a + 1; b < kin; ++b) {
            if (cls[b] >= 0 || level[a] != level[b] || priv[a].size() != priv[b].size() || priv[a].empty()) continue;
            bool ok = true;
            for (int i = 0; i < kin && ok; ++i)
                if (i != a && i != b) ok = w[a][i] == w[b][i];
            int sg[SH_KMAX];
            for (int i = 0; i < kin; ++i) sg[i] = swapped(i, a, b);
            for (int q = 0; q < ng && ok; ++q) {
                const int im = image(q, sg);
                ok = im >= 0 && (owner[q] == a || owner[q] == b || im == q);
            }
            if (ok) c.push_back(b);
        }
        if (c.size() > 1) {
            for (int x : c) cls[x] = static_cast<int>(classes.size());
            classes.push_back(c);
        }
    }
    // a member's private groups in the order of the first member's
    for (auto& c : classes)
        for (int x : c) {
            std::vector<int> m;
            for (int q : priv[c[0]]) {
                int sg[SH_KMAX];
                for (int i = 0; i < kin; ++i) sg[i] = swapped(i, c[0], x);
                m.push_back(x == c[0] ? q : image(q, sg));
            }
            priv[x] = m;
        }
    // automorphisms up to orders of twins: permutations of the groups
    std::vector<std::vector<int>> H;
    int sigma[SH_KMAX], used = 0;
    bool many = false;
    auto search = [&](auto&& self, int i) -> void {
        if (many) return;
        if (i == kin) {
            std::vector<int> pi(ng);
            for (int q = 0; q < ng; ++q)
                if ((pi[q] = image(q, sigma)) < 0) return;
            H.push_back(pi);
            many = H.size() > 32;
            return;
        }
        for (int j = 0; j < kin; ++j) {
            if ((used >> j) & 1 || (i < 2) != (j < 2) || level[i] != level[j]) continue;
            if ((cls[i] < 0) != (cls[j] < 0) || priv[i].size() != priv[j].size()) continue;
            bool ok = true;
            for (int t = 0; t < i && ok; ++t) {
                ok = w[i][t] == w[j][sigma[t]];
                // twins go to twins in increasing order
                if (cls[i] >= 0 && cls[t] == cls[i]) ok = ok && cls[sigma[t]] == cls[j] && sigma[t] < j;
            }
            if (!ok) continue;
            sigma[i] = j;
            used |= 1 << j;
            self(self, i + 1);
            used &= ~(1 << j);
        }
    };
    search(search, 0);
    if (many || H.empty()) return;
    // the symmetries' order: what listing saves at most, beside a factor 2 of the flip
    double order = static_cast<double>(H.size());
    for (const auto& c : classes)
        for (size_t i = 2; i <= c.size(); ++i) order *= static_cast<double>(i);
    if (n_tuple > 1024 && order < (kin > 10 ? 2.0 : 16.0)) return;
    // a tuple as one word, group q's digit in nibble q
    auto digit = [](uint64_t t, int q) { return static_cast<int>((t >> (4 * q)) & 15u); };
    auto block = [&](uint64_t t, int x) {   // a twin's digits
        uint64_t b = 0;
        for (int q : priv[x]) b = b << 4 | static_cast<uint64_t>(digit(t, q));
        return b;
    };
    auto set_block = [&](uint64_t& t, int x, uint64_t b) {
        for (size_t i = priv[x].size(); i-- > 0; b >>= 4) {
            const int q = priv[x][i];
            t = (t & ~(uint64_t{15} << (4 * q))) | (b & 15u) << (4 * q);
        }
    };
    auto sort_twins = [&](uint64_t t) {
        uint64_t b[SH_KMAX];
        for (const auto& c : classes) {
            for (size_t i = 0; i < c.size(); ++i) {
                const uint64_t x = block(t, c[i]);
                size_t j = i;
                for (; j > 0 && b[j - 1] > x; --j) b[j] = b[j - 1];
                b[j] = x;
            }
            for (size_t i = 0; i < c.size(); ++i) set_block(t, c[i], b[i]);
        }
        return t;
    };
    // every qubit of the groups 1: the flip of t is full - t, nibble by nibble, and keeps the signs
    uint64_t full = 0;
    for (int q = 0; q < n_real; ++q) full |= static_cast<uint64_t>(grp[q].m) << (4 * q);
    const uint64_t digits = n_real < 16 ? (uint64_t{1} << (4 * n_real)) - 1 : ~uint64_t{0};
    uint64_t t = 0;
    std::vector<uint64_t> seen;
    double total = 0.0;
    int bits = 0;
    for (const ShellGroup& q : grp) bits += q.m;
    for (uint64_t i = 0; i < n_tuple; ++i) {
        if (i)
            for (int q = 0;; ++q) {
                if (digit(t, q) < grp[q].m) {
                    t += uint64_t{1} << (4 * q);
                    break;
                }
                t &= ~(uint64_t{15} << (4 * q));
            }
        bool sorted = true;
        for (const auto& c : classes)
            for (size_t i = 1; i < c.size() && sorted; ++i) sorted = block(t, c[i - 1]) <= block(t, c[i]);
        if (!sorted) continue;
        seen.clear();
        bool least = true;
        for (const auto& pi : H) {
            uint64_t im = 0;
            for (int q = 0; q < ng; ++q) im |= static_cast<uint64_t>(digit(t, q)) << (4 * pi[q]);
            uint64_t fl = full;   // groups map to groups of their size
            fl = sort_twins((fl - (im & digits)) | (im & ~digits));
            im = sort_twins(im);
            if (im < t || fl < t) {
                least = false;
                break;
            }
            if (std::find(seen.begin(), seen.end(), im) == seen.end()) seen.push_back(im);
            if (std::find(seen.begin(), seen.end(), fl) == seen.end()) seen.push_back(fl);
        }
        if (!least) continue;
        double n = static_cast<double>(seen.size());
        for (const auto& c : classes) {   // arrangements of the members' blocks
            double a = 1.0;
            int run = 1;
            for (size_t i = 1; i < c.size(); ++i) {
                run = block(t, c[i]) == block(t, c[i - 1]) ? run + 1 : 1;
                a *= static_cast<double>(i + 1) / run;
            }
            n *= a;
        }
        ShellCfg e{};
        for (int q = 0; q < ng; ++q) {
            const ShellGroup& G = grp[q];
            if (q >= n_real) {
                for (int j = 0; j < SH_H; ++j)
                    if (G.h[j] && digit(t, q)) e.z |= 1u << (j + 2);
                continue;
            }
            double b = 1.0;
            for (int i = 0; i < digit(t, q); ++i) b = b * (G.m - i) / (i + 1);
            n *= b;
            e.c0 += digit(t, q) * G.wsum;
            for (int i = 0; i < SH_H; ++i) e.h[i] = static_cast<int16_t>(e.h[i] + (G.m - 2 * digit(t, q)) * G.h[i]);
        }
        e.w = std::round(n);
        total += e.w;
        out.push_back(e);
    }
    if (total != std::ldexp(1.0, bits)) {
        out.clear();
        return;
    }
}

int32_t ShellPlanner::find(uint64_t h) {
    if (2 * (shapes_.size() + 1) > table_.size()) {
        std::vector<std::pair<uint64_t, int32_t>> old;
        old.swap(table_);
        table_.assign(std::max<size_t>(64, 4 * old.size()), {0, -1});
        for (const auto& e : old)
            if (e.second >= 0) {
                size_t i = e.first & (table_.size() - 1);
                while (table_[i].second >= 0) i = (i + 1) & (table_.size() - 1);
                table_[i] = e;
            }
    }
    size_t i = h & (table_.size() - 1);
    for (; table_[i].second >= 0; i = (i + 1) & (table_.size() - 1))
        if (table_[i].first == h && shapes_[static_cast<size_t>(table_[i].second)].same(s_)) return table_[i].second;
    table_[i] = {h, static_cast<int32_t>(shapes_.size())};
    shapes_.push_back(s_);
    return table_[i].second;
}

namespace {
// Where each qubit of a tree hangs (u and v: -1) and its coupling there; false: no tree.
bool tree_owners(const Cone& c, bool real, int (&owner)[32], double (&w)[32], double& w_uv) {
    const int kin = c.nd[1];
    for (int q = 0; q < c.k; ++q) owner[q] = -1;
    w_uv = 0.0;
    int n = 0;
    for (size_t e = 0; e < c.ea.size(); ++e) {
        const int a = c.ea[e], b = c.eb[e];
        const double x = real ? c.wf[e] : static_cast<double>(c.ew[e]);
        if (x == 0.0 || a >= kin) continue;   // couplings within the shell have no part in the term
        if (b == 1) {
            w_uv = x;
            continue;
        }
        if (owner[b] >= 0 || (b < kin && a > 1)) return false;
        owner[b] = a;
        w[b] = x;
        ++n;
    }
    return n == c.k - 2;
}
}  // namespace

bool tree_cone(const Cone& c, bool real) {
    int owner[32];
    double w[32], w_uv;
    return tree_owners(c, real, owner, w, w_uv);
}

bool ShellPlanner::add_tree(const Cone& c, ShellCone& out) {
    int owner[32];
    double w[32];
    if (!tree_owners(c, real_, owner, w, out.w_uv)) return false;
    const int kin = c.nd[1];
    out.tree = true;
    out.kin = 0;   // one class
    out.br = static_cast<int32_t>(branches.size());
    int at[32] = {};
    for (int r = 0; r < 2; ++r)
        for (int q = 2; q < kin; ++q) {
            if (owner[q] != r) continue;
            ++(r ? out.nv : out.nu);
            at[q] = static_cast<int>(branches.size());
            ShellBranch b;
            b.w = w[q];
            if (!real_ && std::abs(w[q]) <= 3.0) b.code = static_cast<int16_t>((static_cast<int>(w[q]) + 3) * 343);
            branches.push_back(b);
        }
    for (int q = kin; q < c.k; ++q) {
        ShellBranch& b = branches[static_cast<size_t>(at[owner[q]])];
        const double x = std::abs(w[q]);
        ++b.n_leaf;
        if (b.code >= 0) b.code = b.n_leaf > 6 || x > 3.0 ? int16_t{-1} : static_cast<int16_t>(b.code + (x == 1.0 ? 1 : x == 2.0 ? 7 : 49));
    }
    for (int i = 0; i < out.nu + out.nv; ++i) {
        ShellBranch& b = branches[static_cast<size_t>(out.br + i)];
        if (b.code >= 0) continue;
        b.leaf = static_cast<int32_t>(leaf_w.size());
        for (int q = kin; q < c.k; ++q)
            if (at[owner[q]] == out.br + i) leaf_w.push_back(std::abs(w[q]));
    }
    return true;
}

void ShellPlanner::add_one(const Cone& c, ShellCone& out) {
    if (trees_ && add_tree(c, out)) return;
    const int kin = c.nd[p_ - 1], ns = c.k - kin;
    const size_t ne = c.ea.size();
    out.kin = kin;
    out.edge = static_cast<int64_t>(ea.size());
    s_.kin = kin;
    s_.grp.clear();
    std::memset(s_.level, 0, sizeof(s_.level));
    std::memset(s_.w, 0, sizeof(s_.w));
    for (int q = 0, l = 0; q < kin; ++q) {
        while (q >= c.nd[l]) ++l;
        s_.level[q] = static_cast<uint8_t>(l);
    }
    // order within a distance: by the positions of the neighbours before it, then by degree
    uint32_t before[SH_KMAX] = {};
    int32_t deg[32] = {}, pos[32];
    for (size_t e = 0; e < ne; ++e) {
        ++deg[c.ea[e]];
        ++deg[c.eb[e]];
    }
    for (int q = 0; q < c.k; ++q) pos[q] = q;
    for (int lo = 2; lo < kin;) {
        int hi = lo;
        while (hi < kin && s_.level[hi] == s_.level[lo]) ++hi;
        for (size_t e = 0; e < ne; ++e)
            if (c.eb[e] >= lo && c.eb[e] < hi && c.ea[e] < lo) before[c.eb[e]] |= 1u << (31 - pos[c.ea[e]]);
        int order[SH_KMAX];
        for (int q = lo; q < hi; ++q) {   // stable insertion sort
            int j = q - lo;
            for (; j > 0; --j) {
                const int x = order[j - 1];
                if (before[q] != before[x] ? before[q] < before[x] : deg[q] >= deg[x]) break;
                order[j] = x;
            }
            order[j] = q;
        }
        for (int q = lo; q < hi; ++q) pos[order[q - lo]] = q;
        lo = hi;
    }
    int32_t h[32][SH_H];
    std::memset(h, 0, sizeof(h[0]) * static_cast<size_t>(ns));
    uint64_t hash = static_cast<uint64_t>(kin);
    for (size_t e = 0; e < ne; ++e) {
        int32_t a = pos[c.ea[e]], b = pos[c.eb[e]];
        if (a > b) std::swap(a, b);
        if (a >= kin) continue;   // both ends in the shell: no part in the term
        ea.push_back(a);
        eb.push_back(b);
        ew.push_back(c.ew[e]);
        if (b < kin) {
            s_.w[a][b] = s_.w[b][a] = static_cast<int16_t>(c.ew[e]);
            hash += mix64(static_cast<uint64_t>(static_cast<uint32_t>(c.ew[e])) << 16 | static_cast<uint64_t>(a << 8 | b));
        } else {
            h[b - kin][a - 2] = c.ew[e];
        }
    }
    out.n_edges = static_cast<int32_t>(static_cast<int64_t>(ea.size()) - out.edge);
    // leaves: shell qubits with one coupling, at inner qubits that have two or more
    int owner[32];
    std::fill(std::begin(s_.leaf), std::end(s_.leaf), ShellLeaves{});
    s_.zmask = 0;
    out.n_leaf = out.w_leaf = 0;
    int n_of[SH_KMAX] = {};
    for (int q = 0; q < ns; ++q) {
        owner[q] = -1;
        int n = 0, at = 0;
        for (int i = 0; i < SH_H; ++i)
            if (h[q][i]) {
                ++n;
                at = i + 2;
            }
        if (n != 1) continue;
        owner[q] = at;
        ++n_of[at];
    }
    for (int q = 0; q < ns; ++q) {
        const int a = owner[q];
        if (a < 0 || n_of[a] < 2) continue;
        const int x = std::abs(h[q][a - 2]);
        ShellLeaves& L = s_.leaf[a];
        int i = 0;
        while (i < ZL_W && L.m[i] && L.w[i] != x) ++i;
        if (i == ZL_W) {   // too many couplings
            L = ShellLeaves{};
            n_of[a] = 0;
            s_.zmask &= ~(1u << a);
            continue;
        }
        L.w[i] = static_cast<int16_t>(x);
        ++L.m[i];
        s_.zmask |= 1u << a;
    }
    for (int a = 2; a < kin; ++a) {   // by coupling, so that equal leaves compare equal
        ShellLeaves& L = s_.leaf[a];
        for (int i = 1; i < ZL_W; ++i)
            for (int j = i; j > 0 && L.m[j] && L.w[j] < L.w[j - 1]; --j) {
                std::swap(L.w[j], L.w[j - 1]);
                std::swap(L.m[j], L.m[j - 1]);
            }
        for (int i = 0; i < ZL_W; ++i) {
            const uint64_t x = static_cast<uint64_t>(a) << 32 | static_cast<uint64_t>(static_cast<uint16_t>(L.w[i])) << 16 |
                               static_cast<uint16_t>(L.m[i]);
            if (L.m[i]) hash += mix64(~x);
        }
    }
    out.zmask = s_.zmask;
    for (int q = 0; q < ns; ++q) {   // groups sorted by their couplings
        if (owner[q] >= 0 && (s_.zmask >> owner[q] & 1u)) {
            ++out.n_leaf;
            out.w_leaf += h[q][owner[q] - 2];
            continue;
        }
        size_t i = 0;
        int cmp = 1;
        while (i < s_.grp.size() && (cmp = std::memcmp(s_.grp[i].h, h[q], sizeof(h[q]))) < 0) ++i;
        if (i < s_.grp.size() && cmp == 0) {
            s_.grp[i].m += 1;
            continue;
        }
        ShellGroup g;
        g.m = 1;
        std::memcpy(g.h, h[q], sizeof(g.h));
        for (int x : g.h) g.wsum += x;
        s_.grp.insert(s_.grp.begin() + static_cast<std::ptrdiff_t>(i), g);
    }
    uint64_t nc = 1;
    for (const ShellGroup& g : s_.grp) {
        nc *= static_cast<uint64_t>(g.m) + 1;
        uint64_t x = static_cast<uint64_t>(g.m);
        for (int i = 0; i < SH_H; ++i) x = x * 31 + static_cast<uint32_t>(g.h[i]);
        hash += mix64(x);
    }
    out.nc = s_.nc = static_cast<uint32_t>(nc);   // at most 2^28: the shell holds at most 28 qubits
    s_.hash = mix64(hash);
    out.shape = find(s_.hash);
}

void ShellPlanner::add(const std::vector<const Cone*>& cones, std::vector<ShellCone>& out) {
    out.resize(cones.size());
    const size_t n = cones.size();
    const size_t nt = n < 4096 ? 1 : std::min<size_t>({8, std::max(1u, std::thread::hardware_concurrency()), n / 1024});
    if (nt == 1) {
        for (size_t i = 0; i < n; ++i) add_one(*cones[i], out[i]);
        return;
    }
    std::vector<ShellPlanner> part(nt, ShellPlanner(p_, trees_, real_));
    std::atomic<bool> no_mem{false};
    auto work = [&](size_t t) {
        try {
            for (size_t i = t * n / nt; i < (t + 1) * n / nt; ++i) part[t].add_one(*cones[i], out[i]);
        } catch (const std::bad_alloc&) {   // carried to the caller's thread
            no_mem = true;
        }
    };
    Pool pool;
    size_t started = 1;
    while (started < nt && pool.start(work, started)) ++started;
    for (size_t t = started; t < nt; ++t) work(t);   // no more threads: the remaining ranges run here
    work(0);
    pool.join();
    if (no_mem) throw std::bad_alloc();
    for (size_t t = 0; t < nt; ++t) {   // shapes and couplings of the parts, in order
        const int64_t e0 = static_cast<int64_t>(ea.size());
        ea.insert(ea.end(), part[t].ea.begin(), part[t].ea.end());
        eb.insert(eb.end(), part[t].eb.begin(), part[t].eb.end());
        ew.insert(ew.end(), part[t].ew.begin(), part[t].ew.end());
        const int32_t b0 = static_cast<int32_t>(branches.size()), l0 = static_cast<int32_t>(leaf_w.size());
        for (ShellBranch b : part[t].branches) {
            b.leaf += l0;
            branches.push_back(b);
        }
        leaf_w.insert(leaf_w.end(), part[t].leaf_w.begin(), part[t].leaf_w.end());
        std::vector<int32_t> to(part[t].shapes_.size());
        for (size_t i = 0; i < to.size(); ++i) {
            s_ = part[t].shapes_[i];
            to[i] = find(s_.hash);
        }
        for (size_t i = t * n / nt; i < (t + 1) * n / nt; ++i) {
            out[i].edge += e0;
            out[i].br += b0;
            if (!out[i].tree) out[i].shape = to[static_cast<size_t>(out[i].shape)];
        }
    }
}

void ShellPlanner::list() {
    std::vector<Shape*> todo;
    for (Shape& s : shapes_)
        if (!s.listed) todo.push_back(&s);
    std::atomic<size_t> next{0};
    std::atomic<bool> no_mem{false};
    auto work = [&]() {
        for (size_t i; (i = next.fetch_add(1)) < todo.size();) {
            try {
                todo[i]->enumerate();
            } catch (const std::bad_alloc&) {   // carried to the caller's thread
                no_mem = true;
            }
            todo[i]->listed = true;
        }
    };
    // (a thread takes some 30 us to start)
    const size_t nt = std::min<size_t>({8, std::max(1u, std::thread::hardware_concurrency()), todo.size() / 64 + 1});
    Pool pool;
    for (size_t t = 1; t < nt && pool.start(work); ++t) {}   // what they do not take runs here
    work();
    pool.join();
    if (no_mem) throw std::bad_alloc();
}

const std::vector<ShellCfg>* ShellPlanner::configurations(int32_t shape) const {
    const Shape& s = shapes_[static_cast<size_t>(shape)];
    return s.cfg.empty() ? nullptr : &s.cfg;
}

}  // namespace qaoa
