"""Cones with the same qubits on one shared state (GPU): against the FP64 oracle and the members' own forms.

Tolerances of test_gpu_parity.py.  Every cone size of the kernel (5-14 qubits: items of part of a
wave, one wave and several waves, 8 and 16 amplitudes per thread), even and odd depths, integer
and Gaussian couplings; groups next to cones on their own, reduced plans (orbit weights), batches,
and rows too long for LDS (the members' own kernels).
"""
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


def _ring_with_chords(n, seed):
    i = np.arange(n)
    e = {(min(a, b), max(a, b)) for a, b in zip(i, (i + 1) % n)}
    rng = np.random.default_rng(seed)
    while len(e) < n + 3:
        a, b = sorted(rng.choice(n, 2, replace=False))
        e.add((int(a), int(b)))
    return W.Graph("chords%d" % n, n, np.array(sorted(e), np.int32))


@pytest.mark.parametrize("weights", ["unit", "int", "gauss"])
@pytest.mark.parametrize("n", range(5, 15))
def test_every_cone_size(Q, n, weights):
    g = _ring_with_chords(n, n)
    rng = np.random.default_rng(n)
    w = {"unit": None, "int": rng.choice([-1.0, 2.0, 3.0], g.m), "gauss": rng.normal(size=g.m)}[weights]
    for p in (n // 2, n // 2 + 1) if n < 12 else (4 + n % 2,):
        ga, be = W.draw_angles(3, p, 800 + n + p)
        pl, E, zz = check_energy(Q, g, p, ga, be, reduce=False, weights=w, grad=True)
        # per-term gradients take the members' own forms: their weighted sum is the same gradient
        E1, dg, db = pl.energy_grad(dev(ga), dev(be))
        E2, dg2, db2, zz2, tg = pl.energy_grad_terms(dev(ga), dev(be))
        Wt = float(g.m if w is None else np.abs(w).sum())
        assert np.abs(zz2.cpu().numpy() - zz).max() <= ZZ_TOL
        scale = max(dg2.abs().max().item(), db2.abs().max().item(), 1e-3 * Wt)
        assert max((dg - dg2).abs().max().item(), (db - db2).abs().max().item()) <= 1e-4 * scale


def test_reduced_weights_and_two_components(Q):
    # two copies of one graph, orbits over both: the group's weights count both; and a plan where some
    # cones are the whole graph and others are not
    for n, m in ((7, 3), (12, 2)):
        base = W.circulant(n, (1, 2)) if n > 7 else W.complete(n)
        e = np.concatenate([base.edges, base.edges + n]).astype(np.int32)
        swap = np.concatenate([np.arange(n, 2 * n), np.arange(n)])
        gens = np.concatenate([np.concatenate([base.gens(), base.gens() + n], 1), swap[None]]).astype(np.int32)
        g = W.Graph("pair%d" % n, 2 * n, e, None, gens)
        ga, be = W.draw_angles(2, m + 2, 840 + n)
        check_energy(Q, g, m + 2, ga, be, grad=True)
        check_energy(Q, g, m + 2, ga, be, reduce=False, grad=True)
    g = W.random_regular(14, 3, 6)
    for p in (2, 3, 4):
        ga, be = W.draw_angles(3, p, 850 + p)
        check_energy(Q, g, p, ga, be, reduce=False, grad=True)


def test_batches_items_and_replay(Q):
    gs = [W.random_regular(n, 3, n) for n in (6, 8, 10, 12, 14)]
    p = 5
    rng = np.random.default_rng(1)
    ga, be = rng.uniform(0, np.pi, (len(gs), 7, p)), rng.uniform(0, np.pi / 2, (len(gs), 7, p))
    bp = Q.Plan.batch([(g.n, g.edges) for g in gs], p)
    out = bp.energy_grad(dev(ga), dev(be))
    for j, g in enumerate(gs):
        one = Q.Plan(g.n, g.edges, p=p)
        own = one.energy_grad(dev(ga[j]), dev(be[j]))
        few = one.energy_grad(dev(ga[j][2:3]), dev(be[j][2:3]))
        for x, y, z in zip(out, own, few):
            assert (x[j] - y).abs().max().item() <= 1e-11 * g.m and torch.equal(y[2:3], z)
    gt, bt = dev(ga[3]), dev(be[3])
    rep = Q.Plan(gs[3].n, gs[3].edges, p=p, graph=True)
    buf = (torch.empty(7, dtype=torch.float64, device="cuda"), torch.empty_like(gt), torch.empty_like(bt))
    for it in range(4):
        gt.copy_(dev(ga[3] + 0.2 * it))
        rep.energy_grad(gt, bt, out=buf)
        torch.cuda.synchronize()
        want = Q.Plan(gs[3].n, gs[3].edges, p=p).energy_grad(gt, bt)
        torch.cuda.synchronize()
        assert all(torch.equal(x, y) for x, y in zip(buf, want)), it
    assert rep.info()["graph_replays"] == 3


def test_rows_beyond_lds(Q):
    # weights of 9 and p = 120: the phase rows of the shared state would not fit; own kernels, same values
    g = _ring_with_chords(8, 3)
    w = np.full(g.m, 9.0)
    ga, be = W.draw_angles(1, 120, 870)
    check_energy(Q, g, 120, ga, be, reduce=False, weights=w, grad=False)


@pytest.mark.parametrize("n", [6, 9, 12, 14])
def test_weights_of_any_size(Q, n):
    # weights times 2^e at angles over 2^e: the same circuit, so the results times 2^e (energies, dE/dbeta)
    # and 2^2e (dE/dgamma), bit for bit; products of two weights leave the range of FP32
    g = _ring_with_chords(n, 20 + n)
    w = np.random.default_rng(n).normal(size=g.m)
    p = n // 2 + 1
    ga, be = W.draw_angles(3, p, 880 + n)
    E, dg, db = Q.Plan(g.n, g.edges, p=p, weights=w, reduce=False).energy_grad(dev(ga), dev(be))
    assert torch.isfinite(dg).all() and torch.isfinite(db).all()
    for e in (70, 100):
        s = 2.0 ** e
        E1, dg1, db1 = Q.Plan(g.n, g.edges, p=p, weights=w * s, reduce=False).energy_grad(dev(ga / s), dev(be))
        assert torch.equal(E1, E * s) and torch.equal(db1, db * s) and torch.equal(dg1, dg * s * s)


def test_first_call_of_many_groups_is_linear(Q):
    # 5000 and 20000 prisms (9 cones on the same 6 qubits each): four times the work to upload, not sixteen
    import time
    e = [(0, 1), (1, 2), (0, 2), (3, 4), (4, 5), (3, 5), (0, 3), (1, 4), (2, 5)]
    x = torch.full((1, 2), 0.3, dtype=torch.float64, device="cuda")

    def first(n):
        best = float("inf")
        for _ in range(3):
            pl = Q.Plan.batch([(6, e)] * n, 2, reduce=False)
            torch.cuda.synchronize()
            t = time.perf_counter()
            pl.energy(x, x)
            torch.cuda.synchronize()
            best = min(best, time.perf_counter() - t)
            pl.close()
        return best

    first(100)
    assert first(20000) <= 8 * first(5000)   # 5.4 measured; 13.6 with a search of all cones for each group


@pytest.mark.parametrize("few", [False, True])
def test_own_or_shared_by_size_and_items(Q, few):
    # 12, 13 and 14 qubits in one plan: which sizes share their states in a gradient call depends on members
    # and points (13: two fills of the chip, 14 at p = 2: four); the sums against the terms' own forms
    gs = [W.circulant(n, (1, 2, 3)) for n in (12, 13, 14)]
    gens = [None, gs[1].gens() if few else None, None]   # few: three members of 13 qubits
    pl = Q.Plan.batch([(g.n, g.edges, None, x) for g, x in zip(gs, gens)], 2)
    for P in (1, 8, 32):
        ga, be = W.draw_angles(P, 2, 960 + P)
        E, dg, db = pl.energy_grad(dev(ga), dev(be))
        E2, dg2, db2, zz, tg = pl.energy_grad_terms(dev(ga), dev(be))
        for j, g in enumerate(gs):
            assert (E[j] - E2[j]).abs().max().item() <= ZZ_TOL * g.m / 2
            scale = max(dg2[j].abs().max().item(), db2[j].abs().max().item(), 1e-3 * g.m)
            assert max((dg[j] - dg2[j]).abs().max().item(), (db[j] - db2[j]).abs().max().item()) <= 1e-4 * scale
        own = [Q.Plan(g.n, g.edges, p=2, generators=x, tune=2).energy_grad(dev(ga), dev(be)) for g, x in zip(gs, gens)]
        for j, (g, o) in enumerate(zip(gs, own)):
            scale = max(o[1].abs().max().item(), o[2].abs().max().item(), 1e-3 * g.m)
            assert max((dg[j] - o[1]).abs().max().item(), (db[j] - o[2]).abs().max().item()) <= 1e-4 * scale
