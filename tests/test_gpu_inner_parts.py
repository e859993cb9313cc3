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
