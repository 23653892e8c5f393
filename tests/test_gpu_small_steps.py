"""Steps of small systems, whole steps in one workgroup, against the oracle
and against the same steps by the separate kernels (which the timed form
launches one by one), on both sides of the body count where the one gives way
to the other and of the count of steps of one launch."""
import numpy as np
import pytest

import oracle as O
from paper_1404_2324_amd import genga as G
from paper_1404_2324_amd import workloads as W


def _sim(n, n1, free):
    s = W.planetesimals(n, seed_index=40 + n)
    gp = G.default_params(n1=n1, encounter_free=free, cand_per_body=300)
    return s, gp, G.Simulation(s.m, s.x, s.u, gp, coords="helio")


# n1 = 3: no encounters; 250: groups of two from 15 bodies on; 1000: all
# bodies in one group, two and three bodies too.  Tolerance: the same
# operations in the same order, apart only where a compiler contracts them
# differently (1e-16 a step), and the oracle's own BS to its 1e-13: 1e-12, the
# bound of the other tests against the oracle.
@pytest.mark.gpu
@pytest.mark.parametrize("free", [0, 1])
@pytest.mark.parametrize("n1", [3.0, 250.0, 1000.0])
@pytest.mark.parametrize("n", [2, 3, 15, 16, 17])
def test_small_steps_equal_separate_kernels(n, n1, free):
    print("small steps", n, n1, free, flush=True)
    s, gp, a = _sim(n, n1, free)
    _, _, b = _sim(n, n1, free)
    a.step(19)  # a graph of 16 steps and one of 3
    a.check()
    b.step_kernel_us(19)
    b.check()
    sa, sb = a.stats(), b.stats()
    for k in ("steps", "n_enc", "enc_total", "bs_substeps", "kepler_hist", "kepler_iter_max"):
        assert sa[k] == sb[k], k
    xa, va = [t.cpu().numpy() for t in a.state("dem")]
    xb, vb = [t.cpu().numpy() for t in b.state("dem")]
    op = O.params(G=gp.G, m0=gp.m0, dt=gp.dt, n1=gp.n1, n2=gp.n2, pf=gp.pf, bs_tol=gp.bs_tol,
                  bs_max_depth=gp.bs_max_depth, kepler_max_iter=gp.kepler_max_iter,
                  encounter_free=gp.encounter_free)
    o = O.MassiveSim(op, s.m, s.x, s.u, coords="helio")
    st = o.step(19)
    xo, vo = o.x, o.v
    print("enc", sa["enc_total"], st["enc_total"], flush=True)
    assert sa["enc_total"] == st["enc_total"]
    for p, q in ((xa, xb), (va, vb), (xa, xo), (va, vo)):
        d = np.linalg.norm(p - q, axis=1) / np.linalg.norm(q, axis=1)
        print("rel", d.max(), flush=True)
        assert (d <= 1e-12).all()


# Encounter pairs of a step on both sides of the counts at which the grouping
# changes: one pair a lane (11; 61 to 65), four a lane (256; 268).  Pairs, groups and the largest
# group are whole numbers; states as above.
@pytest.mark.gpu
@pytest.mark.parametrize("n,n1", [(300, 30.0), (90, 196.0), (200, 96.0), (300, 115.0), (300, 118.0)])
def test_groups_of_few_and_many_pairs(n, n1):
    print("groups", n, n1, flush=True)
    s, gp, a = _sim(n, n1, 0)
    op = O.params(G=gp.G, m0=gp.m0, dt=gp.dt, n1=gp.n1, n2=gp.n2, pf=gp.pf, bs_tol=gp.bs_tol,
                  bs_max_depth=gp.bs_max_depth, kepler_max_iter=gp.kepler_max_iter)
    o = O.MassiveSim(op, s.m, s.x, s.u, coords="helio")
    for _ in range(4):
        a.step(1)
        a.check()
        sa, so = a.stats(), o.step(1)
        print({k: (sa[k], so[k]) for k in ("n_enc", "n_groups", "max_group", "n_cand")}, flush=True)
        for k in ("n_enc", "n_groups", "max_group", "n_cand"):
            assert sa[k] == so[k], k
        x, v = [t.cpu().numpy() for t in a.state("dem")]
        for p, q in ((x, o.x), (v, o.v)):
            d = np.linalg.norm(p - q, axis=1) / np.linalg.norm(q, axis=1)
            assert (d <= 1e-12).all()
