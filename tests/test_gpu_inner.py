"""Cones evaluated on their inner qubits (GPU): against the FP64 oracle and the layouts without a shell.

Tolerances of test_gpu_parity.py.  The graphs put every number of inner qubits (3 to 10, and 11
on the other side of the edge) next to shells of one group, equal and unequal leaves, leaves of
two inner qubits, an odd number of configurations (its middle one is its own complement) and
couplings of either sign; depths 2 (sums in registers) and 3-9 (sums in LDS); cones above
14 qubits in one and in several units of work; batches, single launches and graph replay.
"""
import numpy as np
import pytest

import workloads as W
from test_gpu_parity import ZZ_TOL, check_energy, dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def Q():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2101_10296_amd as Q
    return Q


def _graph(inner, leaves):
    """Edge (0, 1), `inner` neighbours alternately at 0, 1 and both, leaves[i] leaves at neighbour i,
    one coupling between the first two neighbours and one leaf shared by the first and last."""
    e = [(0, 1)]
    for i in range(inner):
        e += [[(0, 2 + i)], [(1, 2 + i)], [(0, 2 + i), (1, 2 + i)]][i % 3]
    if inner >= 2:
        e.append((2, 3))
    n = 2 + inner
    for i, m in enumerate(leaves):
        for _ in range(m):
            e.append((2 + i, n))
            n += 1
    if inner >= 3:
        e += [(2, n), (1 + inner, n)]
        n += 1
    g = W.Graph("inner%d" % inner, n, np.array(sorted((min(a, b), max(a, b)) for a, b in e), np.int32))
    return g


def _same(a, b, Wt):
    for i, (x, y) in enumerate(zip(a, b)):
        x, y = x.cpu().numpy(), y.cpu().numpy()
        tol = ZZ_TOL * Wt / 2 if i == 0 else 1e-4 * max(np.abs(y).max(), 1e-3 * Wt)
        assert np.abs(x - y).max() <= tol, (i, np.abs(x - y).max(), tol)


@pytest.mark.parametrize("weights", [False, True])
@pytest.mark.parametrize("inner", range(1, 10))
def test_inner_sizes_p2(Q, inner, weights):
    # every cone of a graph of up to 13 nodes against the oracle: kin = inner + 2 for the edge (0, 1)
    leaves = [1] * inner if inner > 6 else [(i % 3) + 1 for i in range(inner)]
    while inner + 2 + sum(leaves) > 13 and max(leaves) > 0:
        leaves[leaves.index(max(leaves))] -= 1
    g = _graph(inner, leaves)
    w = np.random.default_rng(inner).choice([-2.0, -1.0, 1.0, 3.0], g.m) if weights else None
    ga, be = W.draw_angles(3, 2, 700 + inner)
    check_energy(Q, g, 2, ga, be, reduce=False, weights=w, grad=True)


@pytest.mark.parametrize("p,n", [(3, 8), (3, 13), (4, 11), (5, 13), (6, 13), (9, 12)])
def test_depths(Q, p, n):
    # paths (up to p + 1 inner qubits) and a small tree: prefixes of every length per layer
    e = np.stack([np.arange(n - 1), np.arange(1, n)], 1).astype(np.int32)
    ga, be = W.draw_angles(3, p, 720 + p)
    check_energy(Q, W.Graph("path", n, e), p, ga, be, reduce=False, grad=True)
    t = np.array([(0, 1), (0, 2), (0, 3), (1, 4), (2, 5), (2, 6), (5, 7), (5, 8), (8, 9), (9, 10), (9, 11)], np.int32)
    w = np.array([1, -1, 2, 1, 1, 1, -1, 1, 1, 2, 2], float)
    check_energy(Q, W.Graph("tree", 12, t), p, ga, be, reduce=False, weights=w, grad=True)


@pytest.mark.parametrize("p", [2, 3, 4, 5])
def test_rings_and_angle_edges(Q, p):
    # C_n: 2p inner qubits and a shell of two; angles at the switch of the mixer's factorisation
    g = W.circulant(40, (1,))
    ga, be = W.draw_angles(6, p, 740 + p)
    be[0], be[1], be[2] = np.pi / 4, np.pi / 2, 0.0
    ga[1], ga[3] = 0.0, -7.5
    check_energy(Q, g, p, ga, be, grad=True)


@pytest.mark.parametrize("inner,leaves,weights", [(6, 2, False), (6, 3, True), (8, 2, False), (4, 4, True)])
def test_large_shells_in_units(Q, inner, leaves, weights):
    # 15-28-qubit cones: many configurations, several units of work per cone, against the passes over
    # device memory (tune = 2: the fixed default layout of the kernels without a shell)
    g = _graph(inner, [leaves] * inner)
    w = np.random.default_rng(5).choice([-1.0, 1.0, 2.0], g.m) if weights else None
    ga, be = W.draw_angles(2, 2, 760 + inner)
    a = Q.Plan(g.n, g.edges, p=2, weights=w, reduce=False)
    b = Q.Plan(g.n, g.edges, p=2, weights=w, reduce=False, tune=2)
    Wt = float(np.abs(w).sum()) if weights else float(g.m)
    ra, rb = a.energy_grad(dev(ga), dev(be)), b.energy_grad(dev(ga), dev(be))
    _same(ra, rb, Wt)
    assert sum(a.info()["pass_launches"]) < sum(b.info()["pass_launches"])
    # one item per launch, replays and another number of points: the same sums
    plain = Q.Plan(g.n, g.edges, p=2, weights=w, reduce=False, one_cone_at_a_time=True)
    one = a.energy_grad(dev(ga[1:]), dev(be[1:]))
    for x, y, z in zip(ra, plain.energy_grad(dev(ga), dev(be)), one):
        assert torch.equal(x, y) and torch.equal(x[1:], z)


def test_batch_segments_and_replay(Q):
    # several instances in one class: their workgroups read their own angles; units per wave 1-4
    gs = [W.random_regular(n, 3, n) for n in (30, 8, 64, 200, 12)]
    for P in (1, 5):
        rng = np.random.default_rng(P)
        ga, be = rng.uniform(0, np.pi, (len(gs), P, 2)), rng.uniform(0, np.pi / 2, (len(gs), P, 2))
        bp = Q.Plan.batch([(g.n, g.edges) for g in gs], 2)
        out = bp.energy_grad(dev(ga), dev(be))
        for j, g in enumerate(gs):
            own = Q.Plan(g.n, g.edges, p=2).energy_grad(dev(ga[j]), dev(be[j]))
            for x, y in zip(out, own):
                assert (x[j] - y).abs().max().item() <= 1e-12 * g.m
    g = W.random_regular(40, 4, 3)
    ga, be = W.draw_angles(2, 2, 780)
    gt, bt = dev(ga), dev(be)
    rep = Q.Plan(g.n, g.edges, p=2, graph=True, mem_budget_bytes=8 << 30)
    eager = Q.Plan(g.n, g.edges, p=2, mem_budget_bytes=8 << 30)
    out = (torch.empty(2, dtype=torch.float64, device="cuda"), torch.empty_like(gt), torch.empty_like(bt))
    for it in range(4):
        gt.copy_(dev(ga + 0.1 * it))
        rep.energy_grad(gt, bt, out=out)
        torch.cuda.synchronize()
        want = eager.energy_grad(gt, bt)
        torch.cuda.synchronize()
        assert all(torch.equal(x, y) for x, y in zip(out, want)), it
    assert rep.info()["graph_replays"] == 3
