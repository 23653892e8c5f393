"""Groups of more than 8 members with an odd count, whose BS pairs each member's
partners two by two: the lane beside the last member holds a body of no mass at
rest at (1, 0, 0), and nothing that becomes of it may reach the members."""
import numpy as np
import pytest

import oracle as O
from paper_1404_2324_amd import genga as G
from paper_1404_2324_amd import workloads as W


# G m0 = 2 and tau = 2: in the second column, four substeps of 1/2, that body
# stands at the star exactly (1 - 2 (1/2)^2 2 = 0) and is not a number from there on
@pytest.mark.gpu
@pytest.mark.parametrize("n", [9, 10, 11, 15, 17, 63])
def test_odd_group_beside_the_idle_lane(n):
    print("odd group", n, flush=True)
    rng = np.random.default_rng(n)
    m = rng.uniform(1e-9, 2e-9, n)
    a = 50.0 + rng.uniform(0, 2e-2, n)
    lam = 0.02 * np.arange(n)  # 1 apart; the critical radius is 4 |tau| |v|, 1.6
    x, u = W.elements_to_cartesian(2.0 + m, a, np.full(n, 1e-4), rng.uniform(0, 1e-3, n),
                                   np.zeros(n), np.zeros(n), lam)
    gp = G.default_params(m0=2.0, dt=2.0, n2=4.0)
    op = O.params(G=gp.G, m0=gp.m0, dt=gp.dt, n1=gp.n1, n2=gp.n2, pf=gp.pf, bs_tol=gp.bs_tol,
                  bs_max_depth=gp.bs_max_depth, kepler_max_iter=gp.kepler_max_iter)
    o = O.MassiveSim(op, m, x, u, coords="helio")
    main, sep = [G.Simulation(m, x, u, gp, coords="helio") for _ in range(2)]
    batch = G.BatchedSimulation(np.array([0, n]), np.full(1, 2.0), m, x, u, gp, coords="helio")
    st = o.step(2)
    main.step(2)
    sep.step_kernel_us(2)
    batch.step(2)
    s1, s2 = main.stats(), sep.stats()
    print(st, flush=True)
    assert st["n_groups"] == 1 and st["max_group"] == n
    assert s1["n_groups"] == s2["n_groups"] == 1 and s1["max_group"] == s2["max_group"] == n
    for s in (main, sep, batch):
        q = [t.cpu().numpy() for t in s.state("dem")]
        for p, r in ((q[0], o.x), (q[1], o.v)):
            # the bound of the tests beside the oracle
            assert (np.linalg.norm(p - r, axis=1) <= 1e-12 * np.linalg.norm(r, axis=1)).all()
    assert s1["bs_substeps"] == s2["bs_substeps"]
