"""The backward without a cull at the sizes where its launches change, against the
oracle."""

import numpy as np
import pytest

import oracle
from gpu_helpers import case, dev, host, normwise
from paper_2405_20067_amd import inputs

pytestmark = pytest.mark.gpu

TOL_FP32 = 1e-4    # the bar of the other comparisons with the oracle


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


# 16 (8 from 11 dimensions), 4 and 1 waves a Gaussian
@pytest.mark.parametrize("n,q,k", [(n, q, k) for n, q in [(1, 1), (3, 64), (10, 65), (12, 300)]
                                   for k in (511, 512, 2047, 2048, 2050)] +
                         [(3, 4095, 2049), (3, 4096, 2049), (2, 4096, 32767), (2, 4096, 32769)])
def test_many_gaussians_backward(torch_cuda, n, q, k):
    from paper_2405_20067_amd import ngd
    mix, x, _ = case(n, k, q, seed=n + k, sdiag=(2.0, 8.0), soff=0.5)
    g = inputs.gen_grad_out(q, seed=n)
    m = ngd.Mixture(n, k)
    m.update(*(dev(mix[f]) for f in ("mean", "factor", "weight", "colour")))
    got = [host(t) for t in ngd.eval_backward(m, None, dev(x), dev(g))]
    want = oracle.grad(mix["mean"], mix["factor"], mix["weight"], mix["colour"], x, g)
    for name, a, b in zip(("mean", "factor", "weight", "colour"), got, want):
        assert np.all(np.isfinite(a)), name
        assert normwise(a, b) <= TOL_FP32, name
