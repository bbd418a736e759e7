"""Sizes at which one launch would need 2^32 threads or more along x."""

import numpy as np
import pytest

import oracle
from gpu_helpers import host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _mixture(torch, k, at, reach):
    """k Gaussians on a line, spaced 1, with `reach` as their factor; those at
    `at` have a weight."""
    mean = torch.arange(k, device="cuda", dtype=torch.float32).reshape(k, 1)
    factor = torch.full((k, 1), reach, device="cuda")
    weight = torch.zeros(k, device="cuda")
    weight[at] = 0.5
    return mean, factor, weight, torch.full((k, 3), 0.25, device="cuda")


def test_dense_backward(torch_cuda):
    # every Gaussian is a workgroup's or a wave's
    torch = torch_cuda
    from paper_2405_20067_amd import ngd
    k, at = (1 << 24) + 3, [0, 1, 70000, (1 << 24) - 1, 1 << 24, (1 << 24) + 2]
    p = _mixture(torch, k, at, 0.5)
    m = ngd.Mixture(1, k)
    m.update(*p)
    x = torch.tensor([[0.25], [70000.5], [16777214.0]], device="cuda")
    g = torch.ones(3, 3, device="cuda")
    got = [host(t[at]) for t in ngd.eval_backward(m, None, x, g)]
    want = oracle.grad(*(host(t[at]) for t in p), host(x), host(g))
    for name, a, b in zip(("mean", "factor", "weight", "colour"), got, want):
        np.testing.assert_allclose(a, b.reshape(a.shape), rtol=1e-4, atol=1e-30, err_msg=name)


def test_many_tiles(torch_cuda):
    # a tile a query: as many work items
    torch = torch_cuda
    from paper_2405_20067_amd import ngd
    k, q = 8, (1 << 24) + 5
    p = _mixture(torch, k, list(range(k)), 3.0)
    m = ngd.Mixture(1, k)
    m.update(*p)
    x = (torch.arange(q, device="cuda", dtype=torch.float32) * (8.0 / q)).reshape(q, 1)
    c = ngd.Cull()
    prm = ngd.default_params()
    prm.tile, prm.tiling, prm.n_proj, prm.key_proj = 1, 2, 1, 1
    c.build(m, x, np.ones((1, 1), np.float32), prm)
    assert c.stats()["total"] == k * q
    f = ngd.eval_mixture(m, c, x)
    want = ngd.eval_mixture(m, None, x)
    # 8 positive float32 terms, each sum of at most 8 roundings
    assert float((f - want).abs().max()) <= 16 * 2.0**-24 * float(want.max())


def test_many_gaussians(torch_cuda):
    # the interval test's limits take 16 threads a Gaussian
    torch = torch_cuda
    from paper_2405_20067_amd import ngd
    k, q = (1 << 28) + 65, 200
    if torch.cuda.mem_get_info()[0] < (128 << 30):
        pytest.skip("needs 128 GiB")
    mean = (torch.arange(k, device="cuda", dtype=torch.float64) / k).to(torch.float32)
    near = torch.nonzero((mean - 0.5).abs() < 2e-5).flatten()
    p = (mean.reshape(k, 1), torch.full((k, 1), 4e-7, device="cuda"),
         torch.full((k,), 2.0**-8, device="cuda"), torch.full((k, 3), 0.25, device="cuda"))
    m = ngd.Mixture(1, k)
    m.update(*p)
    x = (0.5 + torch.arange(q, device="cuda", dtype=torch.float64) * 2.0**-24).float()
    x = x.reshape(q, 1)
    g = torch.ones(q, 3, device="cuda")
    prm = ngd.default_params()
    prm.n_proj, prm.key_proj = 1, 1
    c = ngd.Cull().build(m, x, np.ones((1, 1), np.float32), prm)
    # what lies within kappa sigma = 4.3 sigma of the one tile's 200 steps
    total = int(((mean >= 0.5 - 4.3 * 4e-7) & (mean <= 0.5 + 199 * 2.0**-24 + 4.3 * 4e-7)).sum())
    assert abs(c.stats()["total"] - total) <= 0.01 * total
    f = host(ngd.eval_mixture(m, c, x))
    got = [host(t[near]) for t in ngd.eval_backward(m, c, x, g)]
    sub = [host(t[near]) for t in p]
    want = oracle.eval_mixture(*sub, host(x))
    # tau = 1e-4 a pair, of at most 2 % of a query's pairs
    np.testing.assert_allclose(f, want, rtol=1e-4, atol=1e-4 * want.max())
    inside = (sub[0][:, 0] > 0.5) & (sub[0][:, 0] < 0.5 + 100 * 2.0**-24)
    for a, b in zip(got, oracle.grad(*sub, host(x), host(g))):
        a, b = a.reshape(near.numel(), -1)[inside], b.reshape(near.numel(), -1)[inside]
        assert np.abs(a - b).max() <= 2e-4 * np.abs(b).max()
