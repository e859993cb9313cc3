"""Cones of at least 26 qubits on 11 to 14 inner qubits (GPU) against the passes over device memory.

tune = 2 plans run the same cones as passes (their terms are pinned by the oracle in
test_gpu_hbm.py and test_gpu_configs.py; the stored oracle terms of 26- and 29-qubit cones there
also check this form).  Tolerances of test_gpu_parity.py.  Every number of inner qubits at depth 2,
listed and decoded configurations, an odd number of them, couplings of either sign; depth 3 with
two and more qubits mixed in layer 2; batches, launches of one item, other numbers of points.
"""
import numpy as np
import pytest

import workloads as W
from test_gpu_inner import _graph, _same
from test_gpu_parity import dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def Q():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2101_10296_amd as Q
    return Q




@pytest.mark.parametrize("weights", [False, True])
@pytest.mark.parametrize("inner,leaves", [(9, [2] * 7 + [1, 1]), (9, [3] * 2 + [1, 2] * 3 + [3]), (10, [1, 2] * 5),
                                          (11, [1] * 9 + [2, 2]), (12, [1] * 11 + [0])])
def test_inner_sizes_p2(Q, inner, leaves, weights):
    g = _graph(inner, leaves)
    w = np.random.default_rng(inner).choice([-2.0, -1.0, 1.0], g.m) if weights else None
    ga, be = W.draw_angles(2, 2, 900 + inner)
    be[1] = [np.pi / 2 - 0.1, 0.3]
    a = Q.Plan(g.n, g.edges, p=2, weights=w, reduce=False)
    b = Q.Plan(g.n, g.edges, p=2, weights=w, reduce=False, tune=2)
    assert 26 <= a.info()["max_k"] <= 30 and a.cone(0)[0] == a.info()["max_k"]
    ra, rb = a.energy_grad_terms(dev(ga), dev(be)), b.energy_grad_terms(dev(ga), dev(be))
    _same(ra[:3], rb[:3], float(g.m if w is None else np.abs(w).sum()))
    za, zb = ra[3].cpu().numpy(), rb[3].cpu().numpy()
    assert np.abs(za - zb).max() <= 2e-5   # both within 1e-5 of the exact terms
    ta, tb = ra[4].cpu().numpy(), rb[4].cpu().numpy()
    assert np.abs(ta - tb).max() <= 2e-4 * max(np.abs(tb).max(), 1.0)
    E, zz = a.energy(dev(ga), dev(be), term_zz=True)
    assert np.abs(zz.cpu().numpy() - zb).max() <= 2e-5


def test_random_regular_p3(Q):
    # random 3-regular n = 40, p = 3: cones of up to 30 qubits, most of them with 13 or 14 inner qubits
    g = W.random_regular(40, 3, 77)
    ga, be = W.draw_angles(2, 3, 920)
    a = Q.Plan(g.n, g.edges, p=3)
    b = Q.Plan(g.n, g.edges, p=3, tune=2, mem_budget_bytes=64 << 30)
    assert a.info()["max_k"] >= 26
    ra = a.energy_grad(dev(ga), dev(be))
    _same(ra, b.energy_grad(dev(ga), dev(be)), float(g.m))
    assert sum(a.info()["pass_launches"]) < sum(b.info()["pass_launches"])
    b.close()
    # energies alone, one point, one item per launch: the same terms
    E, zz = a.energy(dev(ga), dev(be), term_zz=True)
    zg = a.energy_grad_terms(dev(ga), dev(be))[3]
    assert (zz - zg).abs().max().item() <= 2e-6
    big = [m for m in range(g.m) if a.cone(m)[0] >= 26]
    assert len(big) >= 10
    plain = Q.Plan(g.n, g.edges, p=3, one_cone_at_a_time=True)
    zp = plain.energy(dev(ga), dev(be), term_zz=True)[1]
    z1 = a.energy(dev(ga[1:]), dev(be[1:]), term_zz=True)[1]
    assert torch.equal(zp[:, big], zz[:, big]) and torch.equal(z1[0, big], zz[1, big])
    # a batch of two graphs: each instance's own angles
    h = W.random_regular(36, 3, 5)
    rng = np.random.default_rng(2)
    gb, bb = rng.uniform(0, np.pi, (2, 1, 3)), rng.uniform(0, np.pi / 2, (2, 1, 3))
    bp = Q.Plan.batch([(g.n, g.edges), (h.n, h.edges)], 3)
    Eb = bp.energy(dev(gb), dev(bb))
    bp.close()
    for j, x in enumerate((g, h)):
        own = Q.Plan(x.n, x.edges, p=3).energy(dev(gb[j]), dev(bb[j]))
        assert (Eb[j] - own).abs().max().item() <= 1e-6 * x.m


def test_rows_of_opposite_signs(Q):
    # 30 qubits at p = 3, 14 of them inner: the 3-regular tree around an edge with couplings 8 and 9, and
    # with -8 and -9, in one plan.  Its phases span 509 cut values, a cone's 255: rows of the plan's
    # range would not fit beside the state
    e, outer, n = [(0, 1)], [0, 1], 2
    for _ in range(3):
        outer = [(a, b) for i, a in enumerate(outer) for b in (n + 2 * i, n + 2 * i + 1)]
        e, n, outer = e + outer, n + len(outer), [b for _, b in outer]
    w = np.full(len(e), 9.0)
    w[:7] = 8.0
    assert n == 30 and w.sum() == 254
    ga, be = W.draw_angles(1, 3, 930)
    two = Q.Plan.batch([(n, e, w), (n, e, -w)], 3)
    info = two.info()
    assert info["max_k"] == 30 and info["cut_max"] - info["cut_min"] == 508
    out = two.energy_grad(dev(ga), dev(be))
    for j, x in enumerate((w, -w)):
        own = Q.Plan(n, e, p=3, weights=x)
        assert own.cone(0)[0] == 30
        ref = own.energy_grad(dev(ga), dev(be))
        _same([y[j] for y in out], ref, 254.0)
        assert (out[0][j] - ref[0]).abs().max().item() <= 1e-10 * 254
    passes = Q.Plan(n, e, p=3, weights=w, tune=2, mem_budget_bytes=64 << 30)
    _same([y[0] for y in out], passes.energy_grad(dev(ga), dev(be)), 254.0)


def test_more_units_than_a_grid_holds(Q):
    # 14 inner qubits, 16 shell qubits next to two of them each, 16 different pairs: 2^15 configurations in
    # 4096 units of 1024 threads.  1026 such cones exceed the 2^32 threads of a grid
    e, n = [(0, 1)] + [(0, 2 + i) for i in range(6)] + [(1, 8 + i) for i in range(6)], 14
    for lo in (2, 8):
        for a, b in [(a, b) for a in range(6) for b in range(a + 1, 6)][::2]:
            e += [(lo + a, n), (lo + b, n)]
            n += 1
    one = Q.Plan(n, e, p=2, reduce=False)
    assert n == 30 and one.cone(0)[0] == 30 and 1026 * 4096 * 1024 > 2 ** 32
    ga, be = W.draw_angles(1, 2, 940)
    E, zz = one.energy(dev(ga), dev(be), term_zz=True)
    many = Q.Plan.batch([(n, e)] * 1026, 2, reduce=False)
    Em, zm = many.energy(dev(ga), dev(be), term_zz=True)
    assert torch.equal(zm.reshape(1026, -1)[:, 0], zz[0, 0].expand(1026))
    assert (Em - E).abs().max().item() <= 1e-6 * len(e)
