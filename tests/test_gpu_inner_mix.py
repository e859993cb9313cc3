"""Classes of inner-state cones that share a launch (GPU): bit for bit their own launches.

A plan with one_cone_at_a_time launches every unit and every cone's sum of parts by itself, in the
same order: equality is exact.  Classes with and without leaves and with and without parts, one
to three at once, depths 2 and 3, instances with their own angles, and as many points as bring
one class, then all, past the line where classes get launches of their own.
"""
import numpy as np
import pytest

import workloads as W
from test_gpu_parity import dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def Q():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2101_10296_amd as Q
    return Q


def _ladder(n, rungs):
    """A path of n nodes with some chords of length 3 and a leaf here and there."""
    e = {(i, i + 1) for i in range(n - 1)} | {(i, i + 3) for i in rungs}
    m = n
    for i in range(1, n, 3):
        e.add((i, m))
        m += 1
    return W.Graph("ladder", m, np.array(sorted(e), np.int32))


GRAPHS = {"reg4": lambda: W.random_regular(30, 4, 2), "reg3": lambda: W.random_regular(40, 3, 5), "ladder": lambda: _ladder(24, (0, 4, 5, 11, 17))}


@pytest.mark.parametrize("name,p,P", [("reg4", 2, 1), ("reg4", 2, 5), ("reg3", 2, 3), ("ladder", 2, 4), ("ladder", 3, 3)])
def test_same_bits(Q, name, p, P):
    g = GRAPHS[name]()
    ga, be = W.draw_angles(P, p, 1200 + P)
    gt, bt = dev(ga), dev(be)
    a = Q.Plan(g.n, g.edges, p=p, reduce=False, mem_budget_bytes=8 << 30)
    b = Q.Plan(g.n, g.edges, p=p, reduce=False, mem_budget_bytes=8 << 30, one_cone_at_a_time=True)
    assert torch.equal(a.energy(gt, bt), b.energy(gt, bt))
    for x, y in zip(a.energy_grad_terms(gt, bt), b.energy_grad_terms(gt, bt)):
        assert torch.equal(x, y)


def test_points_and_instances(Q):
    g = GRAPHS["reg3"]()
    P = 8000
    ga, be = W.draw_angles(P, 2, 1210)
    a = Q.Plan(g.n, g.edges, p=2, reduce=False)
    full = a.energy_grad_terms(dev(ga), dev(be))
    for n in (2, 300, 1500):
        part = a.energy_grad_terms(dev(ga[:n]), dev(be[:n]))
        for x, y in zip(full, part):
            assert torch.equal(x[:n], y)
    gs = [GRAPHS[k]() for k in ("reg3", "ladder", "reg3")]
    rng = np.random.default_rng(3)
    ga, be = rng.uniform(0, np.pi, (3, 2, 2)), rng.uniform(0, np.pi / 2, (3, 2, 2))
    out = Q.Plan.batch([(x.n, x.edges) for x in gs], 2).energy_grad(dev(ga), dev(be))
    for j, x in enumerate(gs):
        for u, v in zip(out, Q.Plan(x.n, x.edges, p=2).energy_grad(dev(ga[j]), dev(be[j]))):
            assert (u[j] - v).abs().max().item() <= 1e-12 * x.m
