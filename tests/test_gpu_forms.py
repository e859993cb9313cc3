"""Cones in two forms (GPU): on their inner qubits, or whole, by the number of points of the call.

Small cones run whole from some thousand workgroups on, cones in several rounds of configurations
while they are few.  Against the oracle and the plans with tune = 2, whose cones are all whole (the
same kernel: the same bits), in each form; plans of several graphs, members of shared states,
launches of one item, replay and the allocation-free call.  Tolerances of test_gpu_parity.py.
"""
import ctypes

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


def _path(n):
    return W.Graph("path%d" % n, n, np.stack([np.arange(n - 1), np.arange(1, n)], 1).astype(np.int32))


def _chords(n, seed):
    i = np.arange(n)
    e = {(min(a, b), max(a, b)) for a, b in zip(i, (i + 1) % n)}
    rng = np.random.default_rng(seed)
    while len(e) < n + 3:
        a, b = sorted(rng.choice(n, 2, replace=False))
        e.add((int(a), int(b)))
    return W.Graph("chords%d" % n, n, np.array(sorted(e), np.int32))


def _ladder(n):
    e = [(i, i + 1) for i in range(n - 1)] + [(n + i, n + i + 1) for i in range(n - 1)] + [(i, n + i) for i in range(n)]
    return W.Graph("ladder%d" % n, 2 * n, np.array(sorted(e), np.int32))


def _grads_close(a, b, Wt):
    scale = max(b[1].abs().max().item(), b[2].abs().max().item(), 1e-3 * Wt)
    assert (a[0] - b[0]).abs().max().item() <= ZZ_TOL * Wt / 2
    assert max((a[1] - b[1]).abs().max().item(), (a[2] - b[2]).abs().max().item()) <= 1e-4 * scale


@pytest.mark.parametrize("graph,p,points", [("path13", 3, 3000), ("path13", 5, 5000), ("chords12", 2, 3000), ("chords16", 2, 4000)])
def test_many_points_of_small_cones(Q, graph, p, points):
    g = _path(13) if graph == "path13" else _chords(int(graph[6:]), int(graph[6:]))
    ga, be = W.draw_angles(points, p, 1500 + p)
    pl, _, _ = check_energy(Q, g, p, ga[:3], be[:3], reduce=False, grad=True)   # inner
    whole = Q.Plan(g.n, g.edges, p=p, reduce=False, tune=2)
    few = pl.energy(dev(ga[:3]), dev(be[:3]), term_zz=True)[1]
    zz, zw = (x.energy(dev(ga), dev(be), term_zz=True)[1] for x in (pl, whole))
    assert (zz[:3] - few).abs().max().item() <= 2 * ZZ_TOL and (zz - zw).abs().max().item() <= 2 * ZZ_TOL
    same = [m for m in range(g.m) if torch.equal(zz[:, m], zw[:, m])]   # in the kernel for whole cones
    assert {pl.cone(m)[0] for m in same} and max(pl.cone(m)[0] for m in same) <= 10
    assert not any(torch.equal(few[:, m], zw[:3, m]) for m in same)
    out = pl.energy_grad(dev(ga), dev(be))
    _grads_close(out, whole.energy_grad(dev(ga), dev(be)), float(g.m))
    tg = pl.energy_grad_terms(dev(ga), dev(be))
    _grads_close(tg[:3], out, float(g.m))
    # as launches timed by size, and in a plan of two graphs, its own angles for each
    for x, y in zip(Q.Plan(g.n, g.edges, p=p, reduce=False, profile=True).energy_grad(dev(ga), dev(be)), out):
        assert (x - y).abs().max().item() <= 1e-10 * g.m
    h = _path(11)
    two = Q.Plan.batch([(g.n, g.edges), (h.n, h.edges)], p, reduce=False)
    gb = np.stack([ga, ga[::-1]])
    bb = np.stack([be, be[::-1]])
    rb = two.energy_grad(dev(gb), dev(bb))
    _grads_close([x[0] for x in rb], out, float(g.m))
    _grads_close([x[1] for x in rb], Q.Plan(h.n, h.edges, p=p, reduce=False, tune=2).energy_grad(dev(gb[1]), dev(bb[1])), float(h.m))


@pytest.mark.parametrize("graph,p,size", [("c40", 3, 14), ("ring", 5, 12), ("chords14", 4, 14), ("regular16", 3, 14),
                                          ("ladder16", 3, None)])   # None: its sizes share one inner launch
def test_few_items_of_many_rounds(Q, graph, p, size):
    g = {"c40": lambda: W.circulant(40, (1, 2)), "ring": lambda: W.circulant(60, (1,)), "chords14": lambda: _chords(14, 14),
         "ladder16": lambda: _ladder(16), "regular16": lambda: W.random_regular(16, 3, 5)}[graph]()
    kw = dict(generators=g.gens()) if graph in ("c40", "ring") else dict(reduce=False)
    ga, be = W.draw_angles(2, p, 1520 + p)
    pl = Q.Plan(g.n, g.edges, p=p, **kw)
    whole = Q.Plan(g.n, g.edges, p=p, tune=2, **kw)
    a, b = pl.energy_grad_terms(dev(ga), dev(be)), whole.energy_grad_terms(dev(ga), dev(be))
    _grads_close(a[:3], b[:3], float(g.m))
    assert (a[3] - b[3]).abs().max().item() <= 2 * ZZ_TOL
    assert (a[4] - b[4]).abs().max().item() <= 2e-4 * max(b[4].abs().max().item(), 1.0)
    same = {pl.cone(m)[0] for m in range(pl.n_orbits) if pl.cone(m)[0] <= 14 and torch.equal(a[4][:, :, m], b[4][:, :, m])}
    other = {pl.cone(m)[0] for m in range(pl.n_orbits) if not torch.equal(a[4][:, :, m], b[4][:, :, m])}
    assert (size in same and size not in other) if size else 14 in other
    out = pl.energy_grad(dev(ga), dev(be))
    _grads_close(out, b[:3], float(g.m))
    plain = Q.Plan(g.n, g.edges, p=p, one_cone_at_a_time=True, **kw)
    for x, y in zip(plain.energy_grad_terms(dev(ga), dev(be)), a):
        assert torch.equal(x, y)
    gt, bt = dev(ga), dev(be)
    rep = Q.Plan(g.n, g.edges, p=p, graph=True, **kw)
    buf = (torch.empty(2, dtype=torch.float64, device="cuda"), torch.empty_like(gt), torch.empty_like(bt))
    for it in range(3):
        gt.copy_(dev(ga + 0.1 * it))
        rep.energy_grad(gt, bt, out=buf)
        torch.cuda.synchronize()
        assert all(torch.equal(x, y) for x, y in zip(buf, pl.energy_grad(gt, bt))), it


def test_allocation_free_call_in_the_same_form(Q):
    from paper_2101_10296_amd import _capi
    for g, p, P in ((_path(13), 3, 3000), (W.circulant(60, (1,)), 5, 1)):
        ga, be = W.draw_angles(P, p, 1540 + p)
        gt, bt = dev(ga), dev(be)
        pl = Q.Plan(g.n, g.edges, p=p, generators=None if g.n == 13 else g.gens())
        want = pl.energy_grad(gt, bt)
        got = (torch.zeros(P, dtype=torch.float64, device="cuda"), torch.zeros_like(gt), torch.zeros_like(bt))
        st = _capi.lib().qaoa_energy_grad_noalloc(pl._h, ctypes.c_int64(P), *[ctypes.c_void_p(x.data_ptr()) for x in (gt, bt, *got)],
                                                  ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
        assert st == 0
        torch.cuda.synchronize()
        for x, y in zip(got, want):
            assert (x - y).abs().max().item() <= 1e-12 * g.m


# Whole cones' cut tables are made in parts of 256 entries, fewer to a cone where cones are many: cones of 2 p + 2
# qubits of a small ring and of thousands (workgroups that make a table alone), the same bits.
@pytest.mark.parametrize("p,n", [(2, 300), (3, 700), (4, 5000), (6, 300), (6, 17000)])
def test_tables_of_few_and_many_cones(Q, p, n):
    ga, be = W.draw_angles(2, p, n + p)
    terms = []
    for m in (4 * p + 8, n):
        g = W.circulant(m, (1,))
        pl = Q.Plan(g.n, g.edges, p=p, reduce=False, tune=2)
        zz = pl.energy(dev(ga), dev(be), term_zz=True)[1]
        edges = np.array(sorted(tuple(e) for e in np.sort(np.asarray(g.edges), 1)))
        inside = (edges[:, 1] == edges[:, 0] + 1) & (edges[:, 0] >= p) & (edges[:, 1] < m - p)   # numbered alike
        terms.append(zz[:, torch.as_tensor(np.flatnonzero(inside), device=zz.device)])
    few, many = terms
    assert few.shape[1] == 2 * p + 7 and many.shape[1] == n - 2 * p - 1
    assert torch.equal(few[:, :1].expand_as(few), few) and torch.equal(few[:, :1].expand_as(many), many)
    g = W.circulant(4 * p + 8, (1,))
    check_energy(Q, g, p, ga, be, reduce=True, plan_kw=dict(tune=2))
