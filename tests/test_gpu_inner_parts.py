"""Plans of few cones with many units (GPU): their sums of parts and weighted sums in one launch.

Bit for bit the launches of a plan with one_cone_at_a_time (same units, same order): one cone in
19 parts, two and three cones in parts and in one unit, a weight unit that is not 1, with and
without the caller's terms; and subsets of a number of points past the line where the classes
get launches of their own.
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


def _graph(kind):
    return W.torus2d(8) if kind == "torus" else W.circulant(40, {"13": (1, 3), "14": (1, 4)}[kind])


@pytest.mark.parametrize("kind", ["torus", "13", "14"])
@pytest.mark.parametrize("unit", [1.0, 0.5])
def test_same_bits(Q, kind, unit):
    g = _graph(kind)
    w = np.full(g.m, unit)
    a = Q.Plan(g.n, g.edges, p=2, weights=w, generators=g.gens())
    b = Q.Plan(g.n, g.edges, p=2, weights=w, generators=g.gens(), one_cone_at_a_time=True)
    for P in (1, 6):
        ga, be = W.draw_angles(P, 2, 1300 + P)
        gt, bt = dev(ga), dev(be)
        assert torch.equal(a.energy(gt, bt), b.energy(gt, bt))
        for x, y in zip(a.energy_grad(gt, bt), b.energy_grad(gt, bt)):
            assert torch.equal(x, y)
        for x, y in zip(a.energy_grad_terms(gt, bt), b.energy_grad_terms(gt, bt)):
            assert torch.equal(x, y)


def test_points(Q):
    g = _graph("torus")
    ga, be = W.draw_angles(7200, 2, 1310)
    a = Q.Plan(g.n, g.edges, p=2, generators=g.gens())
    full = a.energy_grad_terms(dev(ga), dev(be))
    for n in (3, 900):
        for x, y in zip(full, a.energy_grad_terms(dev(ga[:n]), dev(be[:n]))):
            assert torch.equal(x[:n], y)


def test_parts_within_the_memory_budget(Q):
    # 98 cones in several parts each, 3000 points: 223 MB of partial sums beside 12 MB of terms, unless the
    # plan's budget (two 18-qubit items) bounds them; the same bits
    g = W.torus2d(7)
    ga, be = W.draw_angles(3000, 2, 1320)
    gt, bt = dev(ga), dev(be)
    out = (torch.empty(3000, dtype=torch.float64, device="cuda"), torch.empty_like(gt), torch.empty_like(bt))
    tight = Q.Plan(g.n, g.edges, p=2, reduce=False, mem_budget_bytes=4 << 20)
    tight.energy_grad(gt[:1], bt[:1])
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    tight.energy_grad(gt, bt, out=out)
    torch.cuda.synchronize()
    assert free - torch.cuda.mem_get_info()[0] < 32 << 20
    for x, y in zip(out, Q.Plan(g.n, g.edges, p=2, reduce=False).energy_grad(gt, bt)):
        assert torch.equal(x, y)


def test_room_for_less_than_a_point(Q):
    # 15 qubits, 10 of them inner, 16 configurations in two parts: 3500 such cones hold 280 KB of gradient
    # sums a point, and the budget one 15-qubit item of 256 KB
    e, n = [(0, 1)] + [(0, 2 + i) for i in range(4)] + [(1, 6 + i) for i in range(4)], 10
    for a, b in [(2, 3), (3, 6), (4, 7), (5, 9), (2, 8)]:
        e += [(a, n), (b, n)]
        n += 1
    w = np.random.default_rng(5).choice([1.0, 2.0, 3.0], len(e))
    ga, be = W.draw_angles(2, 2, 1330)
    item = 2 * (8 << 14) + 2 * 5 * 8
    many = [(n, e, w)] * 1750 + [(n, e, -w)] * 1750
    tight = Q.Plan.batch(many, 2, reduce=False, mem_budget_bytes=item)
    assert tight.info()["max_k"] == 15 and 3500 * 2 * 5 * 8 > item
    free = Q.Plan.batch(many, 2, reduce=False)
    for x, y in zip(tight.energy_grad(dev(ga), dev(be)), free.energy_grad(dev(ga), dev(be))):
        assert torch.equal(x, y)
    with pytest.raises(Q.QaoaError) as ei:
        Q.Plan.batch(many[:1], 2, reduce=False, mem_budget_bytes=item - 1).energy_grad(dev(ga), dev(be))
    assert ei.value.status == Q.QAOA_ENOMEM
