"""Small plans whose calls are one launch (GPU): bit for bit the sums of the separate launches.

A plan with one_cone_at_a_time runs every unit, the parts of a cone and the weighted sums in
launches of their own, in the same order: equality is exact.  Every number of inner qubits
from 3 to 10, one to sixteen units, cones in one and in several parts, depths 2 (sums in
registers) and 3-9 (sums in LDS), a weight unit that is not 1, 1 and many points, with and
without the caller's terms; and plans just beyond the limits.
"""
import numpy as np
import pytest

import workloads as W
from test_gpu_parity import check_energy, dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def Q():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2101_10296_amd as Q
    return Q


def _path(n):
    return W.Graph("path", n, np.stack([np.arange(n - 1), np.arange(1, n)], 1).astype(np.int32))


CASES = [("ring", 40, p, True) for p in (2, 3, 4, 5)] + [
    ("path", 5, 2, False), ("path", 17, 2, False), ("path", 18, 2, False), ("path", 17, 3, False), ("path", 12, 9, False),
    ("path", 17, 6, False), ("steps12", 60, 2, True), ("steps123", 60, 2, True), ("steps15", 80, 2, True)]


@pytest.mark.parametrize("kind,n,p,reduce", CASES)
def test_one_launch(Q, kind, n, p, reduce):
    g = _path(n) if kind == "path" else W.circulant(n, {"ring": (1,), "steps12": (1, 2), "steps123": (1, 2, 3), "steps15": (1, 5)}[kind])
    ws = [None] if reduce else [None, 0.25 * np.random.default_rng(n).choice([-2.0, -1.0, 1.0, 3.0], g.m)]
    if reduce:
        ws.append(np.full(g.m, 0.5))
    for w in ws:
        a = Q.Plan(g.n, g.edges, p=p, weights=w, reduce=reduce)
        b = Q.Plan(g.n, g.edges, p=p, weights=w, reduce=reduce, one_cone_at_a_time=True)
        for P in (1, 7):
            ga, be = W.draw_angles(P, p, 900 + P)
            be[0, 0], ga[P - 1, 0] = np.pi / 4, -7.5
            gt, bt = dev(ga), dev(be)
            assert torch.equal(a.energy(gt, bt), b.energy(gt, bt))
            for x, y in zip(a.energy(gt, bt, term_zz=True), b.energy(gt, bt, term_zz=True)):
                assert torch.equal(x, y)
            for x, y in zip(a.energy_grad(gt, bt), b.energy_grad(gt, bt)):
                assert torch.equal(x, y)
            for x, y in zip(a.energy_grad_terms(gt, bt), b.energy_grad_terms(gt, bt)):
                assert torch.equal(x, y)


def test_against_oracle_and_replay(Q):
    g = W.circulant(13, (1, 2))
    ga, be = W.draw_angles(5, 2, 950)
    check_energy(Q, g, 2, ga, be, grad=True)
    gt, bt = dev(ga), dev(be)
    rep, eager = Q.Plan(g.n, g.edges, p=2, graph=True), Q.Plan(g.n, g.edges, p=2)
    out = (torch.empty(5, dtype=torch.float64, device="cuda"), torch.empty_like(gt), torch.empty_like(bt))
    for it in range(4):
        gt.copy_(dev(ga + 0.1 * it))
        rep.energy_grad(gt, bt, out=out)
        torch.cuda.synchronize()
        assert all(torch.equal(x, y) for x, y in zip(out, eager.energy_grad(gt, bt))), it
    assert rep.info()["graph_replays"] == 3
