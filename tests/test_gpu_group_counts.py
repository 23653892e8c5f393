"""The grouping at the pair counts where it changes, made exactly: one pair a
lane up to 64, four a lane up to 256, the general form beyond, in the form of
main mode and in that of test-particle mode's planets."""
import numpy as np
import pytest

import oracle as O
from paper_1404_2324_amd import genga as G
from paper_1404_2324_amd import workloads as W


def _rings(sizes, seed=5):
    """Groups of bodies 0.006 rad apart, thirteen groups to a circle and the
    circles 0.1 apart from 0.6 on: only members of a group are inside their
    critical radii (0.4 |tau| |v|, below 0.033), and all of a group of up to 3."""
    rng = np.random.default_rng(seed)
    n = sum(sizes)
    m = rng.uniform(1e-10, 2e-10, n)
    g = np.repeat(np.arange(len(sizes)), sizes)
    i = np.concatenate([np.arange(s) for s in sizes])
    a = 0.6 + 0.1 * (g // 13)
    lam = (g % 13) * 2 * np.pi / 13 + 0.006 * i / a ** 1.5
    x, u = W.elements_to_cartesian(1.0 + m, a + rng.uniform(0, 1e-4, n), np.full(n, 1e-4),
                                   rng.uniform(0, 1e-4, n), np.zeros(n), np.zeros(n), lam)
    p = rng.permutation(n)  # pairs in no order
    return m[p], x[p], u[p]


def _op(gp):
    return O.params(G=gp.G, m0=gp.m0, dt=gp.dt, n1=gp.n1, n2=gp.n2, pf=gp.pf, bs_tol=gp.bs_tol,
                    bs_max_depth=gp.bs_max_depth, kepler_max_iter=gp.kepler_max_iter)


def _close(a, b):
    d = np.linalg.norm(a - b, axis=1) / np.linalg.norm(b, axis=1)
    print("rel", d.max(), flush=True)
    return (d <= 1e-12).all()


@pytest.mark.gpu
@pytest.mark.parametrize("pairs,sizes", [(1, [2]), (63, [2] * 63), (64, [2] * 64), (65, [2] * 65),
                                         (129, [3] * 43), (255, [3] * 85), (256, [3] * 85 + [2]),
                                         (257, [3] * 85 + [2, 2]), (320, [2] * 320)])
def test_grouping_at_exact_pair_counts(pairs, sizes):
    print("pairs", pairs, flush=True)
    m, x, u = _rings(sizes)
    gp = G.default_params(cand_per_body=64)
    sim = G.Simulation(m, x, u, gp, coords="helio")
    o = O.MassiveSim(_op(gp), m, x, u, coords="helio")
    for _ in range(3):
        sim.step(1)
        sim.check()
        s, st = sim.stats(), o.step(1)
        assert s["n_enc"] == st["n_enc"] == pairs
        assert s["n_groups"] == st["n_groups"] == len(sizes)
        assert s["max_group"] == max(sizes) and s["n_cand"] == st["n_cand"]
        xg, vg = (t.cpu().numpy() for t in sim.state("dem"))
        assert _close(xg, o.x) and _close(vg, o.v)


# planets all inside each other's critical radii: one group, n (n - 1) / 2 pairs,
# beside particles that meet none of them
@pytest.mark.gpu
@pytest.mark.parametrize("n", [9, 23, 24, 32])
def test_planets_of_test_particle_mode_all_meeting(n):
    print("planets", n, flush=True)
    rng = np.random.default_rng(n)
    m = rng.uniform(1e-13, 2e-13, n)
    lam = 0.02 / n * np.arange(n)
    x, u = W.elements_to_cartesian(1.0 + m, np.full(n, 1.0), np.full(n, 1e-4),
                                   rng.uniform(0, 1e-4, n), np.zeros(n), np.zeros(n), lam)
    at = np.linspace(2.0, 3.0, 300)
    xt, ut = W.elements_to_cartesian(1.0, at, np.zeros(300), np.zeros(300), np.zeros(300),
                                     np.zeros(300), np.linspace(0, 6, 300))
    gp = G.default_params(cand_per_body=64)
    sim = G.TestParticleSimulation(m, x, u, xt, ut, gp, coords="helio")
    o = O.MassiveSim(_op(gp), m, x, u, coords="helio")
    for _ in range(3):
        sim.step(1)
        sim.check()
        s, st = sim.stats(), o.step(1)
        assert s["n_enc"] == st["n_enc"] == n * (n - 1) // 2
        assert s["n_groups"] == st["n_groups"] == 1 and s["max_group"] == n
        xg, vg = (t.cpu().numpy() for t in sim.split_state("dem")[:2])
        assert _close(xg, o.x) and _close(vg, o.v)
