"""Refinement beside the next step, with particles that it removes and particles
that meet a planet again in the step that it makes them late for: particles
aimed at the planets from many distances, so that they pass one after another
through the steps of a graph, against the same steps one call at a time."""
import numpy as np
import pytest

from paper_1404_2324_amd import genga as G
from paper_1404_2324_amd import workloads as W

STEPS = 21  # a graph of 16 (its last step has no branch of its own) and one of 5


def _system(ntp, seed):
    """Half of the particles on orbits, half aimed: 0.02 to 0.4 AU before a planet
    at relative speeds of 0.2 to 1, so that they reach it 0.3 to 30 steps later;
    planets 60 times their size, so that the aim of the far ones is good enough
    for some."""
    p, xt, ut = W.test_particles(ntp=ntp // 2, nplanets=6, seed_index=seed)
    r = W.tp_radii(p.m, ntp)
    r[:6] *= 60
    parts = [W.tp_flybys(p, r, (ntp - ntp // 2) // 8 + 1, seed_index=seed + k, d0=d0, bmax=2.0)
             for k, d0 in enumerate((0.02, 0.04, 0.07, 0.1, 0.15, 0.2, 0.3, 0.4))]
    xt = np.concatenate([xt] + [a for a, _ in parts])[:ntp]
    ut = np.concatenate([ut] + [b for _, b in parts])[:ntp]
    return p, xt, ut, r


def _run(p, xt, ut, r, calls):
    sim = G.TestParticleSimulation(p.m, p.x, p.u, xt, ut, G.default_params(), coords="helio",
                                   radii=r)
    met = []
    for n in calls:
        sim.step(n)
        sim.check()
        met.append(sim.tp_encounters()[0])
    x, v = (t.cpu().numpy() for t in sim.state())
    return x, v, sim.stats(), met, sim.collisions()


@pytest.mark.gpu
# the last: a queue of more than 1024, which the late pass takes 64 to a wave
@pytest.mark.parametrize("ntp,seed", [(8192, 61), (9001, 71), (60000, 81)])
def test_overlap_with_removals(ntp, seed):
    print("tp overlap removal", ntp, seed, flush=True)
    s = _system(ntp, seed)
    x, v, st, met, col = _run(*s, [16, STEPS - 16])
    x1, v1, st1, met1, col1 = _run(*s, [1] * STEPS)
    # passages that need more than the whole-step attempt, particles that meet a
    # planet in two steps running, removals in steps that have a step after them
    # in their graph
    twice = sum(len(np.intersect1d(a[:, 0], b[:, 0])) for a, b in zip(met1[:14], met1[1:15]))
    early = int(((col1["step"] != 15) & (col1["step"] != STEPS - 1)).sum())
    print("enc", st1["tp_enc_total"], "sub", st1["bs_substeps"], "twice", twice, "removed", early,
          "of", st1["tp_removed"], flush=True)
    assert st1["bs_substeps"] > 2 * st1["tp_enc_total"] > 0
    assert twice > 50 and early > 20 and len(np.unique(col1["step"])) > 5
    for k in ("steps", "tp_enc", "tp_enc_total", "tp_removed", "bs_substeps", "kepler_hist",
              "kepler_iter_max"):
        assert st[k] == st1[k], k
    assert np.array_equal(met[0], met1[15]) and np.array_equal(met[1], met1[-1])
    for k in ("tp", "planet", "step", "frac"):
        assert np.array_equal(col[k], col1[k]), k
    # the same step code on both sides; 1e-9 as for the same comparison without
    # removals: rounding (1e-16) that a passage amplifies
    assert np.abs(col["xv"] - col1["xv"]).max() <= 1e-9 * np.abs(col1["xv"]).max()
    gone = np.isnan(x1)
    assert gone.any() and np.array_equal(np.isnan(x), gone)
    for a, b in ((x, x1), (v, v1)):
        d = np.linalg.norm(np.where(gone, 0, a - b), axis=1)
        assert (d <= 1e-9 * np.linalg.norm(np.where(gone, 1, b), axis=1)).all()
