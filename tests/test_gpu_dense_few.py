"""The forward without a cull at the sizes where its launches change, against the
oracle."""

import numpy as np
import pytest

import oracle
from gpu_helpers import case, dev, host, normwise

pytestmark = pytest.mark.gpu

TOL_FP32 = 1e-4    # the bar of the other comparisons with the oracle


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


@pytest.mark.parametrize("k", [1, 15, 16, 17])
@pytest.mark.parametrize("n,q", [(1, 1), (4, 255), (4, 257), (10, 70001), (12, 1023)])
def test_few_gaussians(torch_cuda, n, q, k):
    from paper_2405_20067_amd import ngd
    mix, x, _ = case(n, k, q, seed=n + k, sdiag=(2.0, 8.0), soff=0.5)
    m = ngd.Mixture(n, k)
    m.update(*(dev(mix[f]) for f in ("mean", "factor", "weight", "colour")))
    got = host(ngd.eval_mixture(m, None, dev(x)))
    want = oracle.eval_mixture(mix["mean"], mix["factor"], mix["weight"], mix["colour"], x)
    assert normwise(got, want) <= TOL_FP32


# a wave per 64 queries, 4 and 16 waves sharing the Gaussians; in one dimension
# four queries a lane
@pytest.mark.parametrize("n,q,k", [(2, (1 << 19) - 1, 63), (2, 1 << 19, 63), (2, 1 << 19, 64),
                                   (9, (1 << 17) - 1, 256), (9, 1 << 17, 256),
                                   (10, (1 << 16) - 1, 256), (10, 1 << 16, 256),
                                   (10, 1000, 255), (10, 1000, 256), (1, (1 << 16) - 1, 257),
                                   (1, 1 << 16, 257), (1, (1 << 18) + 5, 64),
                                   (1, (1 << 20) + 300, 65), (1, (1 << 20) + 300, 63)])
def test_launches(torch_cuda, n, q, k):
    test_few_gaussians(torch_cuda, n, q, k)


# records of 4 MiB and one more: two or four queries a lane
@pytest.mark.parametrize("k", [10485, 10486])
@pytest.mark.parametrize("q", [(1 << 15) - 1, 1 << 15, (1 << 16) + 3, (1 << 18) + 65])
def test_large_records(torch_cuda, q, k):
    from paper_2405_20067_amd import ngd
    n = 12
    mix, x, _ = case(n, k, q, seed=q, sdiag=(2.0, 8.0), soff=0.5)
    m = ngd.Mixture(n, k)
    m.update(*(dev(mix[f]) for f in ("mean", "factor", "weight", "colour")))
    got = host(ngd.eval_mixture(m, None, dev(x)))
    at = np.unique(np.r_[0, q - 1, np.random.default_rng(k).integers(0, q, 300)])
    want = oracle.eval_mixture(mix["mean"], mix["factor"], mix["weight"], mix["colour"], x[at])
    assert normwise(got[at], want) <= TOL_FP32


@pytest.mark.parametrize("q", [100, 1 << 17])
def test_partial_sums(torch_cuda, q):
    # Gaussians of value 1 at every query, whose colours add up without rounding
    # within each wave's range but not over the ranges: the sum of the partial
    # sums is rounded once
    from paper_2405_20067_amd import ngd
    n, k = 2, 256
    waves = 16 if q < 1 << 17 else 4
    zero = np.zeros((k, n), np.float32)
    factor = np.tile(np.array([1.0, 0.0, 1.0], np.float32), (k, 1))
    colour = np.ones((k, 3), np.float32) * np.float32(waves / k)   # a partial sum of 1 ...
    colour[:k // waves] *= np.float32(2.0**24)                     # ... the first one 2^24
    m = ngd.Mixture(n, k)
    m.update(dev(zero), dev(factor), dev(np.ones(k, np.float32)), dev(colour))
    got = host(ngd.eval_mixture(m, None, dev(np.zeros((q, n), np.float32))))
    assert np.all(got == np.float32(2.0**24 + waves - 1))
