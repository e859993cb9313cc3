"""Depth-2 trees in closed form (GPU) against the FP64 oracle.

Every cone of a tree graph with a shell is evaluated in FP64: terms and gradients agree with the
oracle to 1e-11 (some 500 operations on values of order one; the angles are below 8 and the
couplings below 8, so phases lose at most 2^6 ulp), far below an FP32 kernel's 1e-7.  Integer
couplings with and without a code (above 3, seven leaves), real ones, more kinds of branches
than a workgroup keeps, up to 8 neighbours, one orbit and more than the one-launch limit,
with and without terms, batches with their own angles, subsets of the points and single
launches bit for bit.
"""
import numpy as np
import pytest

import oracle
import workloads as W
from test_gpu_parity import dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
TOL = 1e-11


@pytest.fixture(scope="module")
def Q():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2101_10296_amd as Q
    return Q


def _tree(n, seed, most):
    """Random tree whose nodes have at most `most` neighbours."""
    rng = np.random.default_rng(seed)
    deg, e = np.zeros(n, int), []
    for i in range(1, n):
        j = rng.choice(np.flatnonzero(deg[:i] < most))
        e.append((j, i))
        deg[j] += 1
        deg[i] += 1
    return W.Graph("tree", n, np.array(sorted(e), np.int32))


def _weights(kind, m, seed):
    rng = np.random.default_rng(seed)
    return {"unit": lambda: None, "spin": lambda: rng.choice([-1.0, 1.0], m), "small": lambda: 0.5 * rng.choice([-3.0, -2.0, 1.0, 3.0], m),
            "large": lambda: rng.choice([-7.0, 4.0, 1.0, 5.0], m), "gauss": lambda: rng.normal(size=m)}[kind]()


def _in_form(g, cone_k):
    """Orbits (edges) whose cone has a shell and at most 10 inner qubits."""
    adj = [set() for _ in range(g.n)]
    for a, b in g.edges.tolist():
        adj[a].add(b)
        adj[b].add(a)
    out = []
    for m, (a, b) in enumerate(g.edges.tolist()):
        inner = adj[a] | adj[b]
        out.append(len(inner) <= 10 and cone_k(m) > len(inner))
    return np.array(out)


@pytest.mark.parametrize("kind", ["unit", "spin", "small", "large", "gauss"])
@pytest.mark.parametrize("n,most", [(12, 3), (14, 5), (13, 8), (40, 3), (300, 3)])
def test_trees(Q, kind, n, most):
    g = _tree(n, n + most, most)
    w = _weights(kind, g.m, n)
    ga, be = W.draw_angles(3, 2, 1100 + n)
    be[0, 0], ga[1, 0] = np.pi / 4, 0.0
    pl = Q.Plan(g.n, g.edges, p=2, weights=w, reduce=False)
    form = _in_form(g, lambda m: pl.cone(m)[0])
    assert form.sum() >= g.m // 2
    E, dg, db, zz, dz = (t.cpu().numpy() for t in pl.energy_grad_terms(dev(ga), dev(be)))
    ref = oracle.plan(g.n, g.edges, w, None, 2, reduce=False)
    Eo, dgo, dbo, zzo = oracle.energy_grad(ref, ga, be)
    assert np.abs(zz - zzo)[:, form].max() <= TOL
    if form.all():
        S = float(np.abs(w).sum()) if w is not None else float(g.m)
        assert np.abs(E - Eo).max() <= TOL * S
        assert max(np.abs(dg - dgo).max(), np.abs(db - dbo).max()) <= 20 * TOL * S
    # each term's own gradient by central differences of its FP64 value
    h = 1e-5
    for d in range(4):
        gp, gm, bp, bm = ga.copy(), ga.copy(), be.copy(), be.copy()
        if d < 2:
            gp[:, d] += h
            gm[:, d] -= h
        else:
            bp[:, d - 2] += h
            bm[:, d - 2] -= h
        hi = pl.energy(dev(gp), dev(bp), term_zz=True)[1].cpu().numpy()
        lo = pl.energy(dev(gm), dev(bm), term_zz=True)[1].cpu().numpy()
        fd = (hi - lo) / (2 * h)
        # third derivatives are below (4 sum |w|)^3 / 6 h^2 with sum |w| <= 8 * 17 couplings in a cone
        assert np.abs(fd - dz[:, d])[:, form].max() <= 2e-4, d


@pytest.mark.parametrize("kind", ["unit", "large", "gauss"])
@pytest.mark.parametrize("n,P", [(30, 1), (30, 700), (257, 5), (258, 5), (600, 300)])
def test_same_bits(Q, kind, n, P):
    g = _tree(n, n, 3)
    w = _weights(kind, g.m, n)
    ga, be = W.draw_angles(P, 2, 1150)
    gt, bt = dev(ga), dev(be)
    a = Q.Plan(g.n, g.edges, p=2, weights=w, reduce=False)
    got, grad = a.energy_grad_terms(gt, bt), a.energy_grad(gt, bt)
    last = a.energy_grad_terms(gt[P - 1:], bt[P - 1:])
    for x, y in zip(got, last):
        assert torch.equal(x[P - 1:], y)
    assert torch.equal(a.energy(gt, bt), grad[0])
    if P <= 5 and n <= 258:
        b = Q.Plan(g.n, g.edges, p=2, weights=w, reduce=False, one_cone_at_a_time=True)
        for x, y in zip(got, b.energy_grad_terms(gt, bt)):
            assert torch.equal(x, y)
        for x, y in zip(grad, b.energy_grad(gt, bt)):
            assert torch.equal(x, y)


def test_batch(Q):
    gs = [_tree(n, n, 3) for n in (20, 700, 9)]
    for kind in ("spin", "gauss"):
        ws = [_weights(kind, g.m, g.n) for g in gs]
        rng = np.random.default_rng(1)
        ga, be = rng.uniform(0, np.pi, (3, 4, 2)), rng.uniform(0, np.pi / 2, (3, 4, 2))
        out = Q.Plan.batch([(g.n, g.edges, w) for g, w in zip(gs, ws)], 2).energy_grad(dev(ga), dev(be))
        for j, (g, w) in enumerate(zip(gs, ws)):
            own = Q.Plan(g.n, g.edges, p=2, weights=w).energy_grad(dev(ga[j]), dev(be[j]))
            for x, y in zip(out, own):
                assert (x[j] - y).abs().max().item() <= 1e-12 * g.m * 10
