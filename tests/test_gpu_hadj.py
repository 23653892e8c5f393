"""GPU reverse-mode gradient of the hybrid step (Eq. 7 with the changeover,
the encounter groups and their BS integration) against the oracle: the
forward map, the full gradient and directional derivatives from the
oracle's complex-step derivative of the main-mode step (every decision held
fixed), and central differences through the GPU forward map.  Systems are
packed so that most pairs sit inside their changeover zone and several
groups form every step.  Tolerances: states 1e-12 relative; gradients 1e-9
of the largest component and directional derivatives 1e-9 (both sides
accumulate thousands of rounding steps through close encounters, whose
Jacobians amplify them)."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_1404_2324_amd import genga as G
from paper_1404_2324_amd import workloads as W

pytestmark = pytest.mark.gpu


def _say(*a):
    print(*a, flush=True)


def _systems(nsys, nplanets=6, seed_index=7, heavy=False, wide=False):
    """heavy: masses log-uniform in [1e-6, 1e-5] (the Hill term of Eq. 6 sets
    the radii), the planets spread wider so that BS converges; wide: the
    wider spread alone (no system of the 1024-system workload fails in 64
    steps)."""
    kw = dict(da=0.03, dphase=0.3) if (heavy or wide) else {}
    m, x, u = W.encounter_systems(nsys=nsys, nplanets=nplanets, seed_index=seed_index, **kw)
    if heavy:
        m = np.exp(np.random.default_rng(seed_index).uniform(np.log(1e-6), np.log(1e-5), m.shape))
    p = O.params()
    v = np.stack([O.helio_to_dem(p, m[s], u[s]) for s in range(nsys)])
    off = np.arange(0, nplanets * nsys + 1, nplanets, dtype=np.int32)
    return off, np.ones(nsys), m.reshape(-1), x.reshape(-1, 3), v.reshape(-1, 3)


def _sim(off, m0s, m, x, v):
    return G.BatchedSimulation(off, m0s, m, x, v, G.default_params(), coords="dem")


def _rel(a, b):
    return np.abs(a - b).max() / max(np.abs(b).max(), 1e-300)


@pytest.mark.parametrize("heavy", [False, True])
def test_hybrid_forward_matches_oracle(heavy):
    nsys, T, K = 6, 10, 4
    off, m0s, m, x, v = _systems(nsys, heavy=heavy)
    _say("forward: systems", nsys, "steps", T, "heavy", heavy)
    sim = _sim(off, m0s, m, x, v)
    sim.adj_forward(T, K)
    sim.check()
    xT, vT = [t.cpu().numpy() for t in sim.state("dem")]
    p = O.params()
    enc = 0
    for s in range(nsys):
        a, b = off[s], off[s + 1]
        o = O.MassiveSim(p, m[a:b], x[a:b], v[a:b])
        st = o.step(T)
        enc += st["enc_total"]
        assert _rel(xT[a:b], o.x) <= 1e-12, (s, _rel(xT[a:b], o.x))
        assert _rel(vT[a:b], o.v) <= 1e-12, (s, _rel(vT[a:b], o.v))
    assert enc > 0
    _say("encounters over the run", enc)


@pytest.mark.parametrize("heavy", [False, True])
def test_hybrid_gradient_matches_oracle(heavy):
    """Every component of dL/dx0, dL/dv0, dL/dm against the oracle's
    complex-step gradient (one derivative per input coordinate)."""
    nsys, T, K = 3, 9, 4          # ragged last segment: 2 x 4 + 1
    off, m0s, m, x, v = _systems(nsys, nplanets=5, seed_index=8, heavy=heavy)
    rng = np.random.default_rng(61)
    gxT, gvT = rng.standard_normal(x.shape), rng.standard_normal(v.shape)
    sim = _sim(off, m0s, m, x, v)
    sim.adj_forward(T, K)
    gx0, gv0, gm = [t.cpu().numpy() for t in sim.adj_backward(gxT, gvT)]
    sim.check()
    p = O.params()
    worst = 0.0
    for s in range(nsys):
        a, b = off[s], off[s + 1]
        ox, ov, om = O.cs_gradient(p, m[a:b], x[a:b], v[a:b], T, gxT[a:b], gvT[a:b])
        for g, o, what in ((gx0[a:b], ox, "x"), (gv0[a:b], ov, "v"), (gm[a:b], om, "m")):
            err = _rel(g, o)
            worst = max(worst, err)
            assert err <= 1e-9, f"system {s} d/d{what}: {err:.3e}"
    _say("gradient vs oracle worst", worst)


def test_hybrid_directional_derivatives_match_oracle():
    nsys, T, K = 8, 24, 8
    off, m0s, m, x, v = _systems(nsys, nplanets=8, seed_index=9)
    rng = np.random.default_rng(62)
    gxT, gvT = rng.standard_normal(x.shape), rng.standard_normal(v.shape)
    sim = _sim(off, m0s, m, x, v)
    sim.adj_forward(T, K)
    gx0, gv0, gm = [t.cpu().numpy() for t in sim.adj_backward(gxT, gvT)]
    sim.check()
    p = O.params()
    for s in range(nsys):
        a, b = off[s], off[s + 1]
        for k in range(2):
            dx, dv = rng.standard_normal(x[a:b].shape), rng.standard_normal(v[a:b].shape)
            dm = rng.standard_normal(m[a:b].shape) * m[a:b]
            _, _, cx, cv, st = O.cs_massive(p, m[a:b], x[a:b], v[a:b], dm, dx, dv, T)
            lhs = np.sum(gxT[a:b] * cx) + np.sum(gvT[a:b] * cv)
            rhs = np.sum(gx0[a:b] * dx) + np.sum(gv0[a:b] * dv) + np.sum(gm[a:b] * dm)
            rel = abs(lhs - rhs) / max(abs(lhs), 1e-300)
            _say("system", s, "direction", k, "groups", st["n_groups"], "relative", rel)
            assert rel <= 1e-9, (s, k, lhs, rhs)


def test_hybrid_map_autograd_against_finite_differences():
    """L = sum |x_T - x_target|^2 through torch.autograd; central differences
    of the GPU forward map over 6 steps with steps of 1e-7 (on the oracle's
    map the same differences are within 7e-7 of its exact derivative;
    1e-6 leaves a truncation error of ~6e-5, 1e-9 rounding of ~1e-5)."""
    nsys, T = 4, 6
    off, m0s, m, x, v = _systems(nsys, nplanets=6, seed_index=10)
    rng = np.random.default_rng(63)
    xp = x * (1.0 + 1e-6 * rng.standard_normal(x.shape))
    vp = v * (1.0 + 1e-6 * rng.standard_normal(v.shape))
    with torch.no_grad():
        tgt, _ = G.hybrid_map(torch.tensor(xp, device="cuda"), torch.tensor(vp, device="cuda"),
                              torch.tensor(m, device="cuda"), off, m0s, T, 4)
    tgt = tgt.detach().clone()
    x0 = torch.tensor(x, device="cuda", requires_grad=True)
    v0 = torch.tensor(v, device="cuda", requires_grad=True)

    def loss(xa, va):
        xT, _ = G.hybrid_map(xa, va, torch.tensor(m, device="cuda"), off, m0s, T, 4)
        return ((xT - tgt) ** 2).sum()

    L = loss(x0, v0)
    L.backward()
    g = (x0.grad.cpu().numpy(), v0.grad.cpu().numpy())
    with torch.no_grad():
        for k, h in ((0, 1e-7), (1, 1e-7)):
            d = [np.zeros_like(x), np.zeros_like(v)]
            d[k] = rng.standard_normal(d[k].shape)
            args_p = [torch.tensor(b + h * e, device="cuda") for b, e in zip((x, v), d)]
            args_m = [torch.tensor(b - h * e, device="cuda") for b, e in zip((x, v), d)]
            fd = (float(loss(*args_p)) - float(loss(*args_m))) / (2 * h)
            an = float(np.sum(g[k] * d[k]))
            _say("direction", k, "adjoint", an, "fd", fd)
            assert abs(an - fd) <= 1e-5 * max(abs(fd), 1e-30)


def test_hybrid_adjoint_full_workload_sampled():
    """1024 systems x 8 planets (the wider packing: ~140 encounters and ~120
    BS substeps per system), 64 steps with a checkpoint every 16:
    the adjoint's directional derivatives for four systems against the
    oracle's complex-step derivatives, and the final states of the same
    systems against the oracle."""
    nsys, T, K = 1024, 64, 16
    off, m0s, m, x, v = _systems(nsys, nplanets=8, seed_index=7, wide=True)
    rng = np.random.default_rng(64)
    gxT, gvT = rng.standard_normal(x.shape), rng.standard_normal(v.shape)
    sim = _sim(off, m0s, m, x, v)
    sim.adj_forward(T, K)
    xT, vT = [t.cpu().numpy() for t in sim.state("dem")]
    gx0, gv0, gm = [t.cpu().numpy() for t in sim.adj_backward(gxT, gvT)]
    sim.check()
    p = O.params()
    for s in (0, 333, 700, 1023):
        a, b = off[s], off[s + 1]
        dx, dv = rng.standard_normal(x[a:b].shape), rng.standard_normal(v[a:b].shape)
        dm = rng.standard_normal(m[a:b].shape) * m[a:b]
        ox, ov, cx, cv, st = O.cs_massive(p, m[a:b], x[a:b], v[a:b], dm, dx, dv, T)
        assert _rel(xT[a:b], ox) <= 1e-11 and _rel(vT[a:b], ov) <= 1e-11, s
        lhs = np.sum(gxT[a:b] * cx) + np.sum(gvT[a:b] * cv)
        rhs = np.sum(gx0[a:b] * dx) + np.sum(gv0[a:b] * dv) + np.sum(gm[a:b] * dm)
        rel = abs(lhs - rhs) / max(abs(lhs), 1e-300)
        _say("system", s, "encounters", st["enc_total"], "BS substeps", st["bs_substeps"],
             "relative", rel)
        assert rel <= 1e-9, (s, lhs, rhs)


def test_hybrid_ragged_systems_and_groups_over_eight():
    """Systems of 3, 12, 7 and 10 planets in one context, groups of up to 12
    members (over 8: the one-column-at-a-time BS path; up to 8: the
    column-parallel one), 12 steps with a checkpoint every 5: states and
    every gradient component against the oracle."""
    sizes, T, K = (3, 12, 7, 10), 12, 5
    p = O.params()
    ms, xs, vs = [], [], []
    for npl in sizes:
        m, x, u = W.encounter_systems(nsys=1, nplanets=npl, seed_index=20)
        ms.append(m[0])
        xs.append(x[0])
        vs.append(O.helio_to_dem(p, m[0], u[0]))
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    m, x, v = np.concatenate(ms), np.concatenate(xs), np.concatenate(vs)
    rng = np.random.default_rng(65)
    gxT, gvT = rng.standard_normal(x.shape), rng.standard_normal(v.shape)
    sim = _sim(off, np.ones(len(sizes)), m, x, v)
    sim.adj_forward(T, K)
    xT, vT = [t.cpu().numpy() for t in sim.state("dem")]
    gx0, gv0, gm = [t.cpu().numpy() for t in sim.adj_backward(gxT, gvT)]
    sim.check()
    big = 0
    for s in range(len(sizes)):
        a, b = off[s], off[s + 1]
        ox, ov, _, _, st = O.cs_massive(p, m[a:b], x[a:b], v[a:b], None, None, None, T)
        big = max(big, st["max_group"])
        assert _rel(xT[a:b], ox) <= 1e-12 and _rel(vT[a:b], ov) <= 1e-12, s
        cx, cv, cm = O.cs_gradient(p, m[a:b], x[a:b], v[a:b], T, gxT[a:b], gvT[a:b])
        for g, o, what in ((gx0[a:b], cx, "x"), (gv0[a:b], cv, "v"), (gm[a:b], cm, "m")):
            err = _rel(g, o)
            _say("system", s, "size", sizes[s], "d/d" + what, err)
            assert err <= 1e-9, (s, what, err)
    assert big > 8


def test_hybrid_small_systems():
    """Systems of 1, 2 (one encounter pair) and 5 planets: the single body
    (no pairs: the Kepler drift and Sun kicks alone), the pair's BS, and a
    group of five, each against the oracle's full gradient."""
    p = O.params()
    parts = ((1, 30), (2, 38), (5, 30))
    ms, xs, vs = [], [], []
    for npl, seed in parts:
        m, x, u = W.encounter_systems(nsys=1, nplanets=npl, seed_index=seed)
        ms.append(m[0])
        xs.append(x[0])
        vs.append(O.helio_to_dem(p, m[0], u[0]))
    sizes = [q[0] for q in parts]
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    m, x, v = np.concatenate(ms), np.concatenate(xs), np.concatenate(vs)
    T, K = 12, 4
    rng = np.random.default_rng(66)
    gxT, gvT = rng.standard_normal(x.shape), rng.standard_normal(v.shape)
    sim = _sim(off, np.ones(len(sizes)), m, x, v)
    sim.adj_forward(T, K)
    xT, vT = [t.cpu().numpy() for t in sim.state("dem")]
    gx0, gv0, gm = [t.cpu().numpy() for t in sim.adj_backward(gxT, gvT)]
    sim.check()
    for s in range(len(sizes)):
        a, b = off[s], off[s + 1]
        ox, ov, _, _, st = O.cs_massive(p, m[a:b], x[a:b], v[a:b], None, None, None, T)
        assert _rel(xT[a:b], ox) <= 1e-12 and _rel(vT[a:b], ov) <= 1e-12, s
        cx, cv, cm = O.cs_gradient(p, m[a:b], x[a:b], v[a:b], T, gxT[a:b], gvT[a:b])
        for g, o, what in ((gx0[a:b], cx, "x"), (gv0[a:b], cv, "v"), (gm[a:b], cm, "m")):
            err = _rel(g, o)
            _say("system of", sizes[s], "encounters", st["enc_total"], "d/d" + what, err)
            assert err <= 1e-9, (s, what, err)


# one segment per step never fills the store of BS substeps that the replay
# keeps (64); one segment for all steps does, and integrates the groups that
# found no room again: the same substeps, so the same gradient
@pytest.mark.parametrize("ckpt", [1, 17, 96])
def test_hybrid_gradient_independent_of_segments(ckpt):
    print("hybrid segments ckpt", ckpt, flush=True)
    nsys, npl, T = 6, 8, 96
    m, x, u = W.encounter_systems(nsys, npl, seed_index=51)
    off = np.arange(0, nsys * npl + 1, npl, dtype=np.int32)
    args = (off, np.ones(nsys), m.reshape(-1), x.reshape(-1, 3), u.reshape(-1, 3))
    run = G.BatchedSimulation(*args, G.default_params())
    run.step(T)
    assert run.stats()["bs_substeps"] > 64 * nsys
    rng = np.random.default_rng(8)
    gx, gv = rng.standard_normal((2, nsys * npl, 3))
    out = []
    for k in (ckpt, 2):
        sim = G.BatchedSimulation(*args, G.default_params())
        sim.adj_forward(T, k)
        out.append([t.cpu().numpy() for t in sim.adj_backward(gx, gv)])
        sim.check()
    for a, b in zip(*out):
        assert np.abs(a - b).max() <= 1e-12 * np.abs(b).max()
