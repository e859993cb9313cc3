"""Weighted sums of few terms (GPU): the orbits of an instance on one wave, and just beyond.

The energy and gradient of a call are the orbit-weighted sums of the terms that it returns:
to FP64 rounding (64 or 65 products of order one: 1e-13), at 1, 63, 64 and 65 orbits, one
and several instances, and more values than a workgroup holds.
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


def _graph(m, seed):
    """A path with a chord (no tree, so that the terms and their sums are launches of their own)."""
    e = [(i, i + 1) for i in range(m - 1)]
    return W.Graph("chord", m, np.array(sorted(e + [(0, 2)]), np.int32)) if m > 2 else W.Graph("edge", 2, np.array([(0, 1)], np.int32))


@pytest.mark.parametrize("m", [3, 63, 64, 65])
@pytest.mark.parametrize("p,P", [(1, 3), (2, 5), (4, 2)])
def test_sums(Q, m, p, P):
    g = _graph(m, 0)
    w = np.random.default_rng(m).choice([-1.0, 1.0, 2.0], g.m)
    ga, be = W.draw_angles(P, p, 1400 + m)
    # (profile: every kernel group on its own)
    pl = Q.Plan(g.n, g.edges, p=p, weights=w, reduce=False, profile=True)
    E, dg, db, zz, dz = (t.cpu().numpy() for t in pl.energy_grad_terms(dev(ga), dev(be)))
    assert zz.shape[1] == m
    np.testing.assert_allclose(E, ((1 - zz) * w / 2).sum(1), rtol=0, atol=1e-13 * 4 * m)
    np.testing.assert_allclose(dg, -(dz[:, :p] * w).sum(2) / 2, rtol=0, atol=1e-11 * m)
    np.testing.assert_allclose(db, -(dz[:, p:] * w).sum(2) / 2, rtol=0, atol=1e-11 * m)


def test_instances(Q):
    gs = [_graph(m, 1) for m in (20, 9, 30)]
    rng = np.random.default_rng(2)
    ga, be = rng.uniform(0, np.pi, (3, 4, 2)), rng.uniform(0, np.pi / 2, (3, 4, 2))
    out = Q.Plan.batch([(g.n, g.edges) for g in gs], 2).energy_grad(dev(ga), dev(be))
    for j, g in enumerate(gs):
        for x, y in zip(out, Q.Plan(g.n, g.edges, p=2).energy_grad(dev(ga[j]), dev(be[j]))):
            assert (x[j] - y).abs().max().item() <= 1e-12 * g.m
