"""Offsets of lists and of their work items at the sizes where the scans change
their launches (16,384 and 2^20 counts): the tiles' by the lists against the CPU
re-implementation and the colours, the Gaussians' by the gradients against the
oracle."""

import numpy as np
import pytest

import oracle
from gpu_helpers import case, dev, host, normwise, queries_of_gaussians
from paper_2405_20067_amd import inputs

pytestmark = pytest.mark.gpu

TOL_FP32 = 1e-4    # the bar of the other comparisons with the oracle


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


# (from 16,385 tiles some of two items, of 512 candidates each)
@pytest.mark.parametrize("k,q", [(600, 16384), (600, 16385), (520, 20481), (5, 65537),
                                 (3, 1 << 20), (3, (1 << 20) + 1)])
def test_tiles(torch_cuda, k, q):
    from paper_2405_20067_amd import ngd
    rng = np.random.default_rng(q)
    mean = rng.random((k, 1)).astype(np.float32)
    factor = np.geomspace(0.02, 2.0, k).astype(np.float32).reshape(k, 1)
    weight, colour = np.full(k, 0.5, np.float32), rng.random((k, 3)).astype(np.float32)
    x = rng.random((q, 1)).astype(np.float32)
    proj = np.ones((1, 1), np.float32)
    m = ngd.Mixture(1, k)
    m.update(dev(mean), dev(factor), dev(weight), dev(colour))
    p = ngd.default_params()
    p.tile, p.tiling, p.n_proj, p.key_proj = 1, 2, 1, 1
    xd = dev(x)
    c = ngd.Cull()
    want = oracle.cull(mean, factor, x, proj, tau=p.tau, tile=1, key_proj=1, tiling=2)
    for _ in range(2):   # a rebuild in the same buffers gives the same
        got = c.build(m, xd, proj, p).export()
        for f in ("gperm", "tile_off", "cand"):
            np.testing.assert_array_equal(got[f], want[f], err_msg=f)
    counts = np.diff(want["tile_off"])
    assert c.stats() == dict(total=counts.sum(), max_per_tile=counts.max(), ntiles=q)
    f = oracle.eval_lists(mean, factor, weight, colour, x, want["tile_off"],
                          want["gperm"][want["cand"]])
    assert normwise(host(ngd.eval_mixture(m, c, xd)), f) <= TOL_FP32


@pytest.mark.parametrize("k", [16384, 16385, 20481, 65536])
def test_gaussians(torch_cuda, k):
    from paper_2405_20067_amd import ngd
    n, tile, q = 4, 64, 3001
    mix, x, proj = case(n, k, q, seed=k)
    wide = np.linspace(0, k - 1, 30).astype(np.int64)   # of several items
    mix["factor"][wide] *= np.geomspace(1.0, 60.0, 30)[:, None].astype(np.float32)
    g = inputs.gen_grad_out(q, seed=n)
    m = ngd.Mixture(n, k)
    m.update(*(dev(mix[f]) for f in ("mean", "factor", "weight", "colour")))
    p = ngd.default_params()
    p.tile = tile
    xd = dev(x)
    c = ngd.Cull().build(m, xd, proj, p)
    got = [host(t) for t in ngd.eval_backward(m, c, xd, dev(g))]
    exp = c.export()
    sel = np.unique(np.concatenate([wide, exp["gperm"][:20], exp["gperm"][-70:],
                                    np.random.default_rng(k).integers(0, k, 200)]))
    sel = sel.astype(np.int64)
    qoff, qidx = queries_of_gaussians(exp, sel, q, tile)
    want = oracle.grad_lists(mix["mean"], mix["factor"], mix["weight"], mix["colour"], x, g,
                             sel, qoff, qidx)
    for name, a, b in zip(("mean", "factor", "weight", "colour"), got, want):
        assert np.all(np.isfinite(a)), name
        assert normwise(a[sel], b) <= TOL_FP32, name
