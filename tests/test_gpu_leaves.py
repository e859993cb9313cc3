"""Shell qubits next to one inner qubit, averaged as a dephasing (GPU).

Against the FP64 oracle and the kernels for whole cones (tune = 2), at the tolerances of
test_gpu_parity.py: cones whose shell is leaves only (at depth 2 trees, in closed form, or
with coupled neighbours) with every number of leaves, equal and unequal ones, no symmetry (16 signs: two
rounds), u and v swapped, coupled neighbours, couplings of either sign, none of which is
1, and just beyond the limits (couplings above 3, seven leaves, a shared leaf: groups or the
general kernel); larger inner states with leaves at depths 2 to 4; an inner qubit with five
different couplings, which keeps them as groups; rows and workgroups that are not full, several
cones per row, batches, single launches and subsets of the points bit for bit.
"""
import numpy as np
import pytest

import workloads as W
from test_gpu_inner import _same
from test_gpu_parity import check_energy, dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def Q():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2101_10296_amd as Q
    return Q


def _tree(at_u, at_v, leaves, extra=(), shared=None):
    """Edge (0, 1), at_u and at_v further neighbours (2 ..), leaves[i] leaves at neighbour i."""
    e = [(0, 1)] + [(0, 2 + i) for i in range(at_u)] + [(1, 2 + at_u + i) for i in range(at_v)] + list(extra)
    n = 2 + at_u + at_v
    for i, m in enumerate(leaves):
        for _ in range(m):
            e.append((2 + i, n))
            n += 1
    if shared:
        e += [(shared[0], n), (shared[1], n)]
        n += 1
    return W.Graph("tree", n, np.array(sorted((min(a, b), max(a, b)) for a, b in e), np.int32))


TREES = [
    (_tree(1, 1, (1, 1)), [(1,), (2, -1), (3,)]),
    (_tree(1, 1, (6, 3)), [(1,), (3, -3)]),
    (_tree(2, 0, (2, 3)), [(1,), (-2,)]),
    (_tree(2, 1, (2, 2, 2)), [(1,), (1, -1, 2)]),
    (_tree(3, 1, (0, 1, 2, 3)), [(1,), (1, 2, 3, -1)]),
    (_tree(2, 2, (2, 2, 2, 2)), [(1,), (1, -1), (1, 2, 3)]),
    (_tree(2, 2, (1, 2, 2, 1)), [(1,), (2,)]),
    (_tree(2, 2, (2, 2, 2, 1), extra=((2, 3),)), [(1,), (-1, 1)]),
    (_tree(2, 2, (2, 2, 1, 1), extra=((0, 4),)), [(1,)]),
    (_tree(2, 2, (2, 2, 2, 0)), [(4,), (1, 4)]),       # couplings beyond the rows' limit
    (_tree(1, 1, (7, 2)), [(1,)]),                     # seven leaves
    (_tree(2, 2, (2, 2, 1, 1), shared=(2, 4)), [(1,), (1, -1)]),
    (_tree(4, 1, (2, 2, 1, 1, 0)), [(1,), (2, -1)]),   # 7 inner qubits
    (_tree(1, 1, (5, 1)), [(1, 2, 3, 4, 5)]),          # five couplings at one qubit: groups
]


@pytest.mark.parametrize("i", range(len(TREES)))
def test_trees_p2(Q, i):
    g, weights = TREES[i]
    assert g.n <= 14
    for ws in weights:
        w = np.array([ws[j % len(ws)] for j in range(g.m)], float)
        for scale in (1.0, 0.5):
            ga, be = W.draw_angles(3, 2, 1000 + i)
            be[0, 0] = np.pi / 4
            ga[1, 0] = 0.0
            check_energy(Q, g, 2, ga, be, reduce=False, weights=scale * w, grad=True)


@pytest.mark.parametrize("p", [2, 3, 4])
def test_general_kernel(Q, p):
    # paths of trees: up to 10 inner qubits with leaves, against the kernels for whole cones
    e = [(i, i + 1) for i in range(6)]
    n = 7
    for i in range(7):
        for _ in range(2 if i % 2 else 1):
            if n < 14:
                e.append((i, n))
                n += 1
    g = W.Graph("comb", n, np.array(sorted(e), np.int32))
    for w in (np.ones(g.m), np.random.default_rng(p).choice([-3.0, -1.0, 1.0, 2.0], g.m)):
        ga, be = W.draw_angles(4, p, 1050 + p)
        a = Q.Plan(g.n, g.edges, p=p, weights=w, reduce=False)
        b = Q.Plan(g.n, g.edges, p=p, weights=w, reduce=False, tune=2)
        _same(a.energy_grad(dev(ga), dev(be)), b.energy_grad(dev(ga), dev(be)), float(np.abs(w).sum()))


@pytest.mark.parametrize("n,P", [(10, 1), (26, 3), (400, 1), (400, 2000)])
def test_rows_and_units(Q, n, P):
    g = W.random_regular(n, 3, n)
    w = np.random.default_rng(n).choice([-1.0, 1.0], g.m)
    ga, be = W.draw_angles(P, 2, 1070)
    a = Q.Plan(g.n, g.edges, p=2, weights=w, reduce=False)
    got = a.energy_grad_terms(dev(ga), dev(be))
    one = a.energy_grad_terms(dev(ga[P - 1:]), dev(be[P - 1:]))
    for x, y in zip(got, one):
        assert torch.equal(x[P - 1:], y)
    if P <= 3:
        plain = Q.Plan(g.n, g.edges, p=2, weights=w, reduce=False, one_cone_at_a_time=True)
        for x, y in zip(got, plain.energy_grad_terms(dev(ga), dev(be))):
            assert torch.equal(x, y)
        b = Q.Plan(g.n, g.edges, p=2, weights=w, reduce=False, tune=2)
        _same(got[:3], b.energy_grad(dev(ga), dev(be)), float(g.m))
