"""Small systems with several encounter groups in a step, which their one
workgroup integrates side by side (two waves each of two, two for the largest of
three, one each of more), and with one, which takes every wave, against the
separate kernels and the oracle."""
import numpy as np
import pytest

import oracle as O
from paper_1404_2324_amd import genga as G
from paper_1404_2324_amd import workloads as W


def clusters(sizes, seed=3):
    """Groups of bodies 0.008 / a^(1/2) apart on one circle, the circles 0.4
    apart: within a group neighbours are inside their critical radius (0.4 |tau|
    |v|, 0.025 / a^(1/2)), no two groups are.  Masses of 1e-9 keep the passages
    gentle."""
    rng = np.random.default_rng(seed)
    n = sum(sizes)
    m = rng.uniform(1e-9, 2e-9, n)
    a = np.concatenate([np.full(s, 0.9 + 0.4 * k) for k, s in enumerate(sizes)])
    lam = np.concatenate([0.008 * np.arange(s) / (0.9 + 0.4 * k) ** 1.5 + 1.7 * k
                          for k, s in enumerate(sizes)])
    a += rng.uniform(0, 2e-4, n)
    x, u = W.elements_to_cartesian(1.0 + m, a, np.full(n, 1e-4), rng.uniform(0, 1e-3, n),
                                   np.zeros(n), np.zeros(n), lam)
    return m, x, u


# one group; two, three (the largest first, in the middle and last), four, eight (a
# wave takes two); one of more than 8 members beside others, first and last; the
# largest counts of 16 bodies
@pytest.mark.gpu
@pytest.mark.parametrize("sizes", [[2], [8, 8], [2, 2, 2], [3, 5, 4], [7, 3, 3], [3, 3, 6],
                                   [2, 7], [9, 3], [4, 12], [16], [5], [4, 4, 4, 4],
                                   [2, 3, 2, 4, 2], [2] * 8, [9, 2, 2], [2, 2, 12], [10, 3, 3]])
def test_small_system_groups(sizes):
    print("small groups", sizes, flush=True)
    m, x, u = clusters(sizes)
    gp = G.default_params()
    one, many, sep = [G.Simulation(m, x, u, gp, coords="helio") for _ in range(3)]
    op = O.params(G=gp.G, m0=gp.m0, dt=gp.dt, n1=gp.n1, n2=gp.n2, pf=gp.pf, bs_tol=gp.bs_tol,
                  bs_max_depth=gp.bs_max_depth, kepler_max_iter=gp.kepler_max_iter)
    o = O.MassiveSim(op, m, x, u, coords="helio")
    for _ in range(6):
        one.step(1)
        sep.step_kernel_us(1)
        st = o.step(1)
        s1, s2 = one.stats(), sep.stats()
        for k in ("n_enc", "n_groups", "max_group", "n_cand"):
            assert s1[k] == s2[k] == st[k], k
        assert s1["n_groups"] == len(sizes) and s1["max_group"] == max(sizes)
    many.step(6)
    assert one.stats()["bs_substeps"] == sep.stats()["bs_substeps"] == many.stats()["bs_substeps"]
    q = [[t.cpu().numpy() for t in s.state("dem")] for s in (one, many, sep)] + [[o.x, o.v]]
    # the same steps by one launch each and by one launch: nothing between
    # differs; against the others the bound of the tests beside the oracle
    for a, b, tol in ((0, 1, 0.0), (0, 2, 1e-12), (0, 3, 1e-12)):
        for i in range(2):
            d = np.linalg.norm(q[a][i] - q[b][i], axis=1) / np.linalg.norm(q[b][i], axis=1)
            print(a, b, d.max(), flush=True)
            assert (d <= tol).all()
