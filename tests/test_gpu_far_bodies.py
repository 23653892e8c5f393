"""Bodies so far out that a squared or cubed separation overflows: the plain
quotients and roots make such a pair's term zero, and so must the device's
short forms, whose refinement would make it NaN."""
import numpy as np
import pytest

from paper_1404_2324_amd import genga as G


# r^2 in range, just below and above the largest double, far above
@pytest.mark.gpu
@pytest.mark.parametrize("far", [1e100, 1e154, 1.5e154, 1e200])
def test_energy_with_a_far_body(far):
    print("energy far", far, flush=True)
    m = np.array([1e-6, 2e-6, 3e-6])
    x = np.array([[1.0, 0, 0], [0, 2.0, 0], [far, 0, 0]])
    v = np.array([[0, 1.0, 0], [-0.7, 0, 0], [0, 0, 0]])
    sim = G.Simulation(m, x, v, G.default_params(encounter_free=1), coords="dem")
    E, L = sim.energy()
    P = (m[:, None] * v).sum(0)
    Eo = (0.5 * (m * (v ** 2).sum(1)).sum() + 0.5 * (P ** 2).sum() - m[0] / 1.0 - m[1] / 2.0
          - m[2] / far - m[0] * m[1] / np.sqrt(5.0) - m[2] * (m[0] + m[1]) / far)
    # a dozen terms of the size of the largest, each rounded a few times
    assert abs(E - Eo) <= 64 * 2.2e-16 * m[0]
    assert np.isfinite(L).all()


# the same three bodies with and without a fourth one whose r^3 is in range, near
# the largest double, above it
@pytest.mark.gpu
@pytest.mark.parametrize("far", [1e90, 5.5e102, 6e102, 1e120])
def test_hybrid_adjoint_forward_with_a_far_body(far):
    print("hybrid far", far, flush=True)
    m = np.array([1e-6, 2e-6, 3e-6, 1e-9])
    x = np.array([[1.0, 0, 0], [0, 2.0, 0], [0, 0, 3.0], [far, 0, 0]])
    v = np.array([[0, 1.0, 0], [-0.7, 0, 0], [0.5, 0, 0], [0, 0, 0]])
    out = []
    for n in (3, 4):
        sim = G.BatchedSimulation(np.array([0, n]), np.ones(1), m[:n], x[:n], v[:n],
                                  G.default_params(), coords="dem")
        sim.adj_forward(4, 2)
        xT, vT = (t.cpu().numpy() for t in sim.state("dem"))
        sim.check()
        out.append((xT, vT))
    (xa, va), (xb, vb) = out
    # the far body adds less than a rounding to the others
    assert np.abs(xb[:3] - xa).max() <= 1e-15 and np.abs(vb[:3] - va).max() <= 1e-15
    # which it moves by the Sun kick alone, as all bodies
    assert np.linalg.norm(xb[3] - x[3]) <= 1e-15 * far and np.abs(vb[3]).max() <= 1e-15
