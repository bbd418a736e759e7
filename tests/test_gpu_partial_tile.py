"""The last tile of a query count that does not fill it: its 64-query groups
past the end keep nothing, whatever an earlier build in the same handle left in
the buffers.  A rebuild that follows one with more queries and every pair kept
must give the gradients of a fresh handle bit for bit, and a query that is not a
number, the one that lanes past the end repeat, must reach only the Gaussians
that keep its own group."""

import numpy as np
import pytest

import oracle
from gpu_helpers import case, dev, host
from paper_2405_20067_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


@pytest.mark.parametrize("precision", ["FP32", "BF16_MFMA"])
@pytest.mark.parametrize("k", [300, 65537])
@pytest.mark.parametrize("tile,q", [(256, 900), (512, 1100)])
def test_groups_past_the_end(torch_cuda, tile, q, k, precision):
    from paper_2405_20067_amd import ngd
    n, prec = 6, getattr(ngd, precision)
    full = -(-q // tile) * tile
    mix, x, _ = case(n, k, full, seed=k + tile)
    # one projection: many candidates that no group keeps
    proj = inputs.gen_projections(n, 1, seed=3)
    g = inputs.gen_grad_out(full, seed=2)
    p = ngd.default_params()
    p.tile, p.tiling, p.n_proj, p.key_proj = tile, 2, 1, 1
    first = q // tile * tile   # the last tile's first query
    bad = x[:q].copy()
    bad[first, 1] = np.nan
    xf, xb = dev(x), dev(bad)
    gd, gq = dev(g), dev(g[:q])
    m = ngd.Mixture(n, k)
    names = ("mean", "factor", "weight", "colour")
    used = ngd.Cull()
    # Gaussians that reach every query: every flag of every group is set
    m.update(*(dev(mix[f] * np.float32(1000.0 if f == "factor" else 1.0)) for f in names))
    used.build(m, xf, proj, p)
    st = ngd.eval_stats(m, used, xf, precision=prec)
    assert st["kept"] == st["examined"] == k * (full // 64)
    ngd.eval_backward(m, used, xf, gd, precision=prec)
    m.update(*(dev(mix[f]) for f in names))
    used.build(m, xb, proj, p)
    ngd.eval_mixture(m, used, xb, precision=prec)
    got = [host(t) for t in ngd.eval_backward(m, used, xb, gq, precision=prec)]
    fresh = ngd.Cull().build(m, xb, proj, p)
    ngd.eval_mixture(m, fresh, xb, precision=prec)
    want = [host(t) for t in ngd.eval_backward(m, fresh, xb, gq, precision=prec)]
    for name, a, b in zip(names, got, want):
        np.testing.assert_array_equal(a, b, err_msg=name)
    # the Gaussians that keep no other query of the bad one's group, one unit of
    # the squared distance from the threshold
    others = np.arange(first + 1, min(first + 64, q))
    idx = np.arange(k)
    msq = oracle.msq_pairs(mix["mean"], mix["factor"], bad, np.tile(others, k),
                           np.repeat(idx, others.size)).reshape(k, others.size)
    cut = 2.0 * np.log(2.0) * (np.log2(1.0 / p.tau) + 20.0)
    dropped = idx[msq.min(1) > cut + 1.0]
    assert dropped.size > k // 4
    for name, a in zip(names, got):
        assert np.all(np.isfinite(a.reshape(k, -1)[dropped])), name
