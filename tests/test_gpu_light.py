"""The backward of large mixtures, where a Gaussian with a handful of queries
takes its moments in LDS and the others go to work items, against the float64
oracle over the candidate pairs: the smallest size of that rule, ragged tiles
and groups, and Gaussians on both sides of its limits (32 queries of a group, 64
in all, 32 kept entries)."""

import numpy as np
import pytest

import oracle
from gpu_helpers import case, dev, host, normwise, queries_of_gaussians
from paper_2405_20067_amd import inputs

pytestmark = pytest.mark.gpu

K = 65537          # one more than the last size without the rule
TOL_FP32 = 1e-4    # the bar of the other comparisons with the oracle


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


@pytest.mark.parametrize("k", [K, K + 62])
@pytest.mark.parametrize("n,tile,q", [(1, 64, 900), (2, 256, 3001), (3, 192, 2500),
                                      (6, 1024, 2100), (10, 256, 5003), (12, 100, 1777)])
def test_gradients(torch_cuda, n, tile, q, k):
    from paper_2405_20067_amd import ngd
    mix, x, proj = case(n, k, q, seed=n + k)
    # Gaussians of every reach, from one query to all of them, around queries
    wide = np.linspace(0, k - 1, 40).astype(np.int64)
    mix["factor"][wide] *= np.geomspace(1.0, 60.0, 40)[:, None].astype(np.float32)
    mix["mean"][wide] = x[np.random.default_rng(n).integers(0, q, 40)]
    g = inputs.gen_grad_out(q, seed=n)
    m = ngd.Mixture(n, k)
    m.update(*(dev(mix[f]) for f in ("mean", "factor", "weight", "colour")))
    p = ngd.default_params()
    p.tile = tile
    xd = dev(x)
    c = ngd.Cull().build(m, xd, proj, p)
    got = [host(t) for t in ngd.eval_backward(m, c, xd, dev(g))]
    again = [host(t) for t in ngd.eval_backward(m, c, xd, dev(g))]
    for a, b in zip(got, again):
        np.testing.assert_array_equal(a, b)
    exp = c.export()
    # the wide ones, those nearest to a query, both ends, and some of the rest
    rng = np.random.default_rng(k)
    sel = np.unique(np.concatenate([wide, exp["gperm"][:20], exp["gperm"][-70:],
                                    rng.integers(0, k, 300)])).astype(np.int64)
    qoff, qidx = queries_of_gaussians(exp, sel, q, tile)
    want = oracle.grad_lists(mix["mean"], mix["factor"], mix["weight"], mix["colour"], x, g,
                             sel, qoff, qidx)
    for name, a, b in zip(("mean", "factor", "weight", "colour"), got, want):
        assert np.all(np.isfinite(a)), name
        assert normwise(a[sel], b) <= TOL_FP32, name


@pytest.mark.parametrize("where", ["query", "upstream"])
def test_not_a_number(torch_cuda, where):
    # one bad query: the gradients of the Gaussians that keep its group of 64
    # are not numbers, the others' are finite, as by work items
    from paper_2405_20067_amd import ngd
    n, k, q, tile = 6, K, 6000, 256
    mix, x, proj = case(n, k, q, seed=3)
    g = inputs.gen_grad_out(q, seed=1)
    m = ngd.Mixture(n, k)
    m.update(*(dev(mix[f]) for f in ("mean", "factor", "weight", "colour")))
    p = ngd.default_params()
    p.tile = tile
    clean = ngd.Cull().build(m, dev(x), proj, p).export()
    bad = int(clean["perm"][700])
    if where == "query":
        x[bad, 1] = np.nan
    else:
        g[bad, 2] = np.nan
    xd = dev(x)
    c = ngd.Cull().build(m, xd, proj, p)
    got = [host(t) for t in ngd.eval_backward(m, c, xd, dev(g))]
    exp = c.export()
    at = int(np.flatnonzero(exp["perm"] == bad)[0])
    t, grp = at // tile, at % tile // 64
    others = exp["perm"][t * tile + grp * 64:min(t * tile + grp * 64 + 64, q)]
    others = others[others != bad].astype(np.int64)
    cand = exp["gperm"][exp["cand"][exp["tile_off"][t]:exp["tile_off"][t + 1]]].astype(np.int64)
    msq = oracle.msq_pairs(mix["mean"], mix["factor"], x, np.tile(others, cand.size),
                           np.repeat(cand, others.size)).reshape(cand.size, others.size)
    # the threshold in units of the squared distance, one unit off on both sides
    least = msq.min(1) if where == "query" else np.minimum(
        msq.min(1), oracle.msq_pairs(mix["mean"], mix["factor"], x, np.full(cand.size, bad), cand))
    cut = 2.0 * np.log(2.0) * (np.log2(1.0 / p.tau) + 20.0)
    kept, dropped = cand[least < cut - 1.0], np.setdiff1d(np.arange(k), cand[least < cut + 1.0])
    assert kept.size > 0
    # (a bad query's colour gradient is G g: not a number with either)
    for name, a in zip(("mean", "factor", "weight", "colour"), got):
        a = a.reshape(k, -1)
        assert np.all(np.isnan(a[kept]).any(1)), name
        assert np.all(np.isfinite(a[dropped])), name
