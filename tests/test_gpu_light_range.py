"""The backward of large mixtures sums over every query of the kept groups, also
those whose Gaussian value lies below the forward's threshold: an upstream
gradient may be so large there that they make the result."""

import numpy as np
import pytest

import oracle
from gpu_helpers import dev, host

pytestmark = pytest.mark.gpu

TOL_FP32 = 1e-4    # the bar of the other comparisons with the oracle


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


@pytest.mark.parametrize("k", [300, 65537])
@pytest.mark.parametrize("n", [1, 4, 10])
def test_large_upstream_far_out(torch_cuda, n, k):
    from paper_2405_20067_amd import ngd
    rng = np.random.default_rng(n)
    q, tile, at = 128, 128, [5, 17, 200, 299]
    mean = np.full((k, n), 50.0, np.float32)     # far from every query ...
    mean[at] = 0.0                               # ... but for these
    factor = np.zeros((k, n * (n + 1) // 2), np.float32)
    for a in range(n):
        factor[:, a * (a + 1) // 2 + a] = 0.1
    weight = np.full(k, 0.5, np.float32)
    colour = rng.random((k, 3)).astype(np.float32)
    # exponents (base 2) of the Gaussian values: one query keeps the group at
    # 2^-30; the others lie beyond the threshold of 2^-33.3, one of them, at
    # 2^-40 or 2^-60, with an upstream gradient that outweighs it
    e = np.full(q, 200.0)
    e[3], e[20], e[70], e[90] = 30.0, 40.0, 30.0, 60.0
    u = rng.standard_normal((q, n))
    u /= np.linalg.norm(u, axis=1, keepdims=True)
    x = (u * (0.1 * np.sqrt(2.0 * np.log(2.0) * e))[:, None]).astype(np.float32)
    g = rng.standard_normal((q, 3)).astype(np.float32)
    g[20] *= 2.0**16
    g[90] *= 2.0**36
    m = ngd.Mixture(n, k)
    m.update(dev(mean), dev(factor), dev(weight), dev(colour))
    p = ngd.default_params()
    p.tile, p.tiling, p.n_proj, p.key_proj = tile, 2, 1, 1
    # a projection on which the queries' extent reaches the Gaussians
    proj = np.ones((1, n), np.float32)
    xd = dev(x)
    c = ngd.Cull().build(m, xd, proj, p)
    assert c.stats()["total"] >= len(at)
    got = [host(t) for t in ngd.eval_backward(m, c, xd, dev(g))]
    sel = np.array(at, np.int64)
    qoff = np.arange(len(at) + 1, dtype=np.int64) * q
    qidx = np.tile(np.arange(q, dtype=np.int64), len(at))
    want = oracle.grad_lists(mean, factor, weight, colour, x, g, sel, qoff, qidx)
    for name, a, b in zip(("mean", "factor", "weight", "colour"), got, want):
        a, b = a[sel].reshape(len(at), -1), b.reshape(len(at), -1)
        assert np.all(np.abs(a - b).max(1) <= TOL_FP32 * np.abs(b).max(1)), name
