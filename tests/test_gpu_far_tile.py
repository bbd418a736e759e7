"""A tile that reaches further than the filter's scales: one query so far along a
coordinate that the others' offsets from the tile's centre leave the float16
features' range, and Gaussians so wide along it that they do not notice.  The
others' pairs must be kept as anywhere else."""

import numpy as np
import pytest

import oracle
from gpu_helpers import dev, host, normwise

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


@pytest.mark.parametrize("far", [2.0**50, 2.0**59, 2.0**61, -(2.0**62), 2.0**63, 2.0**70])
@pytest.mark.parametrize("n", [2, 5, 10])
def test_far_query(torch_cuda, n, far):
    from paper_2405_20067_amd import ngd
    rng = np.random.default_rng(n)
    k, q, tile = 40, 200, 256
    mean = rng.random((k, n)).astype(np.float32)
    sig = np.full((k, n), 0.2)
    sig[:, n - 1] = 0.2 * 2.0**20
    factor = np.zeros((k, n * (n + 1) // 2), np.float32)
    for a in range(n):
        factor[:, a * (a + 1) // 2 + a] = sig[:, a]
    weight = (0.1 + 0.9 * rng.random(k)).astype(np.float32)
    colour = rng.random((k, 3)).astype(np.float32)
    x = rng.random((q, n)).astype(np.float32)
    x[77, n - 1] = far
    proj = rng.standard_normal((4, n)).astype(np.float32)
    m = ngd.Mixture(n, k)
    m.update(dev(mean), dev(factor), dev(weight), dev(colour))
    p = ngd.default_params()
    p.tile, p.tiling, p.n_proj, p.key_proj = tile, 2, 4, 4
    xd = dev(x)
    c = ngd.Cull().build(m, xd, proj, p)
    assert c.stats()["total"] == k   # every Gaussian is a candidate of the one tile
    want = oracle.eval_mixture(mean, factor, weight, colour, x)
    assert np.abs(want[:64]).min() > 0
    for prec in (ngd.FP32, ngd.BF16_MFMA):
        got = host(ngd.eval_mixture(m, c, xd, precision=prec))
        assert normwise(got, want) <= 1e-4   # the bar of the other comparisons with the oracle
        st = ngd.eval_stats(m, c, xd, precision=prec)
        assert st["kept"] == -(-q // 64) * k
