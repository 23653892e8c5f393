"""The encounter-free adjoint on both sides of the lines at which its layout
changes for systems of one to four bodies: partner lanes, one lane per body with
at most one wave on a SIMD, one lane per body.  Copies of two systems give the
two systems' own results, wherever they sit."""
import numpy as np
import pytest

from test_gpu_adjoint import _grad, _spaced


# waves: 1 body 1024 and 1025; 2 bodies with partner lanes (512), without (257),
# 1024 and 1025; 4 bodies 1024 with partner lanes, 257 without, 1025
@pytest.mark.gpu
@pytest.mark.parametrize("n,copies", [(1, 65536), (1, 65600), (2, 8192), (2, 8194), (2, 32768),
                                      (2, 32800), (4, 4096), (4, 4098), (4, 16400)])
def test_adjoint_layout_lines(n, copies):
    print("adjoint lines", n, copies, flush=True)
    sizes = [n, max(1, n - 1)]
    off, m0s, m, x, v = _spaced(sizes, 80 + n)
    rng = np.random.default_rng(n)
    gx, gv = rng.standard_normal((2,) + x.shape)
    one = _grad(off, m0s, m, x, v, gx, gv, 6, 4)
    r = copies // 2
    big = np.concatenate([[0], np.cumsum(sizes * r)]).astype(np.int32)
    t = [np.tile(q, (r,) + (1,) * (q.ndim - 1)) for q in (m, x, v, gx, gv)]
    many = _grad(big, np.ones(2 * r), *t, 6, 4)
    k = int(off[-1])
    for a, b in zip(one, many):
        for at in (0, (r // 2) * k, (r - 1) * k):
            assert np.abs(b[at:at + k] - a).max() <= 1e-12 * np.abs(a).max()
