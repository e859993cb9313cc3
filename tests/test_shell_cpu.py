"""The leaves' factors of inner qubits (csrc/shell.hpp), compiled for the host (CPU).

A plan without leaves has no leaf records: where its descriptors point, memory holds whatever an
earlier plan left.  Factors are taken for the qubits of the mask alone, so nothing is read there.
"""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2101_10296_amd", "csrc")

PROGRAM = r"""
#include <cmath>
#include <cstdio>
#include "shell.hpp"
using namespace qaoa;
int main() {
    const double t = 0.37;
    double2 ct[6], fac[16];
    for (int j = 0; j < 6; ++j) ct[j] = make_double2(std::cos(j * t), std::sin(j * t));
    for (auto& f : fac) f = make_double2(-7.0, -9.0);
    // no leaves: no record is read, whatever the descriptor holds
    for (int lane = 0; lane < 64; ++lane) z_factors(0u, nullptr, 0, ct, lane, fac);
    for (auto& f : fac)
        if (f.x != -7.0 || f.y != -9.0) return 1;
    // leaves on qubits 3 and 13: the records of the others hold counts and couplings out of any range
    ZLeaf rec[20];
    for (auto& q : rec)
        for (int i = 0; i < ZL_W; ++i) q.w[i] = q.m[i] = 32767;
    rec[4 + 3] = ZLeaf{{1, 5, 0, 0}, {2, 1, 0, 0}};
    rec[4 + 13] = ZLeaf{{2, 0, 0, 0}, {3, 0, 0, 0}};
    for (int lane = 0; lane < 64; ++lane) z_factors(1u << 3 | 1u << 13, rec, 4, ct, lane, fac);
    const double f3 = std::pow(std::cos(t), 2) * std::cos(5 * t);
    const double d3 = -2 * std::cos(t) * std::sin(t) * std::cos(5 * t) - std::pow(std::cos(t), 2) * 5 * std::sin(5 * t);
    const double f13 = std::pow(std::cos(2 * t), 3), d13 = -6 * std::pow(std::cos(2 * t), 2) * std::sin(2 * t);
    for (int i = 0; i < 16; ++i) {
        const double x = i == 3 ? f3 : i == 13 ? f13 : -7.0, y = i == 3 ? d3 : i == 13 ? d13 : -9.0;
        if (std::fabs(fac[i].x - x) > 1e-15 || std::fabs(fac[i].y - y) > 1e-14) return 2;
    }
    // weights over all signs sum to 1, their derivatives to 0
    double s = 0.0, ds = 0.0;
    for (uint32_t z : {0u, 1u << 3, 1u << 13, 1u << 3 | 1u << 13}) {
        double w = 1.0;
        ds += z_weight(1u << 3 | 1u << 13, z, fac, w);
        s += w;
    }
    return std::fabs(s - 1.0) <= 1e-15 && std::fabs(ds) <= 1e-15 ? 0 : 3;
}
"""


def test_factors_read_no_record_of_a_qubit_without_leaves(tmp_path):
    inc = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include")
    if shutil.which("g++") is None or not os.path.isdir(inc):
        pytest.skip("no host compiler or HIP headers")
    src = tmp_path / "leaves.cpp"
    src.write_text(PROGRAM)
    exe = str(tmp_path / "leaves")
    subprocess.run(["g++", "-std=c++17", "-O1", "-w", "-D__HIP_PLATFORM_AMD__", "-I", inc, "-I", CSRC, str(src), "-o", exe],
                   check=True)
    assert subprocess.run([exe]).returncode == 0


ALLOC_PROGRAM = r"""
#include <cstdlib>
#include <new>
#include "inner_plan.hpp"
#include "plan.hpp"
static thread_local long left = -1;   // allocations of this thread until one fails; -1: none does
static bool hit = false;
void* operator new(std::size_t n) {
    if (left >= 0 && left-- == 0) { hit = true; throw std::bad_alloc(); }
    if (void* p = std::malloc(n ? n : 1)) return p;
    throw std::bad_alloc();
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, std::size_t) noexcept { std::free(p); }
using namespace qaoa;
int main() {
    std::vector<Cone> cones(9000);
    for (size_t i = 0; i < cones.size(); ++i) {
        Cone& c = cones[i];   // an edge, two neighbours, two qubits behind them; 90 shapes of them
        c.k = 6;
        c.nodes = {0, 1, 2, 3, 4, 5};
        c.ea = {0, 0, 1, 2, 2, 3};
        c.eb = {1, 2, 3, 4, 5, 4};
        c.ew = {1, 1 + static_cast<int>(i % 9), 1, 1, 1 + static_cast<int>(i % 10), 1};
        c.wf.assign(c.ew.begin(), c.ew.end());
        c.nd[0] = 2;
        c.nd[1] = 4;
        for (int d = 2; d < 10; ++d) c.nd[d] = 6;
    }
    std::vector<const Cone*> at;
    for (const Cone& c : cones) at.push_back(&c);
    int failed = 0;
    for (long n = 0;; ++n) {
        hit = false;
        try {
            ShellPlanner s(2);
            std::vector<ShellCone> out;
            left = n;
            s.add(at, out);
            s.list();
            left = -1;
            if (!s.configurations(out[0].shape)) return 2;
            if (!hit) break;   // fewer allocations than n
        } catch (const std::bad_alloc&) {
            left = -1;
            ++failed;
        }
    }
    if (failed <= 20) return 1;
    // the cones of a ring of 5000 edges: the allocations up to and behind the start of the threads
    std::vector<int32_t> u, v;
    for (int32_t i = 0; i < 5000; ++i) {
        u.push_back(i);
        v.push_back((i + 1) % 5000);
    }
    failed = 0;
    for (long n = 0; n < 300; ++n) {
        try {
            HostPlan hp;
            PlanOptions opt;
            left = n;
            build_host_plan(5000, 5000, u.data(), v.data(), nullptr, 0, nullptr, 1, opt, hp);
            left = -1;
            if (hp.cones.size() != 5000 || hp.cones[4999].k != 4) return 3;
        } catch (const std::bad_alloc&) {
            left = -1;
            ++failed;
        }
    }
    return failed > 20 ? 0 : 4;
}
"""


def test_failed_allocations_end_in_an_exception(tmp_path):
    # every allocation of the planning thread fails once, those that start its threads among them: the caller
    # gets std::bad_alloc or a plan made on fewer threads, the process goes on
    if shutil.which("g++") is None:
        pytest.skip("no host compiler")
    src = tmp_path / "alloc.cpp"
    src.write_text(ALLOC_PROGRAM)
    exe = str(tmp_path / "alloc")
    subprocess.run(["g++", "-std=c++17", "-O1", "-w", "-pthread", "-I", CSRC, str(src), os.path.join(CSRC, "inner_plan.cpp"),
                    os.path.join(CSRC, "plan.cpp"), "-o", exe], check=True)
    assert subprocess.run([exe], timeout=100).returncode == 0
