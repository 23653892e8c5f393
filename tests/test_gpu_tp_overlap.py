"""Test-particle steps of one graph, whose refinement runs beside the next
step, against the same steps one call at a time (nothing beside them), on both
sides of the particle count from which the graph has two branches."""
import numpy as np
import pytest

from paper_1404_2324_amd import genga as G
from paper_1404_2324_amd import workloads as W


def _run(calls, ntp, radii):
    p, xt, ut = W.test_particles(ntp=ntp, nplanets=8, seed_index=33)
    sim = G.TestParticleSimulation(p.m, p.x, p.u, xt, ut, G.default_params(), coords="helio",
                                   radii=radii(p.m, ntp))
    for n in calls:
        sim.step(n)
        sim.check()
    x, v = (t.cpu().numpy() for t in sim.state())
    st = sim.stats()
    return x, v, st, sim.tp_encounters(), sim.collisions()


# 21 steps: a graph of 16 (even last step) and one of 5 (odd)
@pytest.mark.gpu
@pytest.mark.parametrize("ntp", [255, 8191, 8192, 10007])
def test_overlapped_steps_equal_single_steps(ntp):
    print("tp overlap ntp", ntp, flush=True)
    x, v, st, (pr, d2, _), col = _run([21], ntp, W.tp_radii)
    x1, v1, st1, (pr1, d21, _), col1 = _run([1] * 21, ntp, W.tp_radii)
    # the same step code on both sides: every count equal, and states apart by
    # no more than rounding (1e-16) that a passage at 1e-4 of a critical radius
    # 0.2 amplifies by its square
    for k in ("steps", "tp_enc", "tp_enc_total", "tp_removed", "bs_substeps", "kepler_hist",
              "kepler_iter_max"):
        assert st[k] == st1[k], k
    assert np.array_equal(pr, pr1) and np.allclose(d2, d21, rtol=1e-9)
    assert np.array_equal(col["tp"], col1["tp"]) and np.array_equal(col["step"], col1["step"])
    gone = np.isnan(x1)
    assert np.array_equal(np.isnan(x), gone)
    for a, b in ((x, x1), (v, v1)):
        d = np.linalg.norm(np.where(gone, 0, a - b), axis=1)
        n = np.linalg.norm(np.where(gone, 1, b), axis=1)
        assert (d <= 1e-9 * n).all()
