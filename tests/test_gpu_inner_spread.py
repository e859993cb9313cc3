"""A few cones in more than four units (GPU): spread over compute units for few points, a workgroup per
point for many, bit for bit the same and as single launches (same units, same order)."""
import pytest

import workloads as W
from test_gpu_parity import dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("steps", [(1, 2, 3), (1, 5)])
def test_same_bits(steps):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2101_10296_amd as Q
    g = W.circulant(90, steps)
    ga, be = W.draw_angles(700, 2, 1500)
    a = Q.Plan(g.n, g.edges, p=2, generators=g.gens())
    b = Q.Plan(g.n, g.edges, p=2, generators=g.gens(), one_cone_at_a_time=True)
    many = a.energy_grad_terms(dev(ga), dev(be))
    for n in (2, 100, 300):
        for x, y in zip(many, a.energy_grad_terms(dev(ga[:n]), dev(be[:n]))):
            assert torch.equal(x[:n], y)
    for x, y in zip(many, b.energy_grad_terms(dev(ga[:2]), dev(be[:2]))):
        assert torch.equal(x[:2], y)
