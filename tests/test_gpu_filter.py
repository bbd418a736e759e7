"""The culled forward's matrix-core filter at the edges of its ranges: list
lengths around its words, rounds and items, and inputs at the ends of its
scales.  The filter may drop no (64-query group, candidate) pair that comes
below the skip threshold anywhere in the group: the number of pairs kept must
lie between the float64 counts for the threshold moved by 1e-3 either way (the
float32 rounding of the distances it is compared with), and the colours must
meet the float32 bar of 1e-4 over the candidate pairs."""

import math

import numpy as np
import pytest

import oracle
from gpu_helpers import case, dev, host, normwise, per_query_csr

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _run(mix, x, proj, tile, tau):
    from paper_2405_20067_amd import ngd
    k, n = mix["mean"].shape
    q = x.shape[0]
    m = ngd.Mixture(n, k)
    m.update(*(dev(mix[f]) for f in ("mean", "factor", "weight", "colour")))
    p = ngd.default_params()
    p.tile, p.tau = tile, tau
    xd = dev(x)
    c = ngd.Cull().build(m, xd, proj, p)
    exp = c.export()
    qoff, gidx = per_query_csr(exp, q, tile)
    want = oracle.eval_lists(mix["mean"], mix["factor"], mix["weight"], mix["colour"], x, qoff,
                             gidx)
    assert np.abs(want).max() > 0
    for prec in (ngd.FP32, ngd.BF16_MFMA):
        assert normwise(host(ngd.eval_mixture(m, c, xd, precision=prec)), want) <= 1e-4
    # M' of every candidate pair, its smallest over each 64-query group
    qi = np.repeat(np.arange(q), np.diff(qoff))
    msq = oracle.msq_pairs(mix["mean"], mix["factor"], x, qi, gidx) * (0.5 * math.log2(math.e))
    pos = np.empty(q, np.int64)
    pos[exp["perm"]] = np.arange(q)
    per = -(-tile // 64)
    grp = pos[qi] // tile * per + pos[qi] % tile // 64
    key = grp * k + gidx
    order = np.argsort(key, kind="stable")
    first = np.flatnonzero(np.r_[True, np.diff(key[order]) > 0])
    best = np.minimum.reduceat(msq[order], first)
    skip = -math.log2(tau) + 20.0
    st = ngd.eval_stats(m, c, xd)
    lo, hi = (best <= skip * 0.999).sum(), (best <= skip * 1.001).sum()
    print(f"kept {st['kept']} of {st['filtered']} filtered, float64 {lo}..{hi} of {best.size}")
    assert lo <= st["kept"] <= hi


@pytest.mark.parametrize("k", [1, 63, 64, 65, 255, 256, 257, 511, 512, 513, 1030])
@pytest.mark.parametrize("n", [3, 10, 12])
def test_list_lengths(torch_cuda, n, k):
    # a threshold that leaves every Gaussian a candidate of every tile
    mix, x, proj = case(n, k, 150, seed=n + k)
    _run(mix, x, proj, 128, 1e-30)


def _scaled(mix, x, s, shift=0.0):
    f = np.float32
    out = dict(mix, mean=(mix["mean"] * f(s) + f(shift)).astype(f),
               factor=(mix["factor"] * f(s)).astype(f))
    return out, (x * f(s) + f(shift)).astype(f)


@pytest.mark.parametrize("what", ["tiny", "huge", "far", "one-point", "tile-1", "wide-factors",
                                  "mixed-sizes"])
@pytest.mark.parametrize("n", [2, 6, 10])
def test_scales(torch_cuda, n, what):
    tile, tau = 256, 1e-4
    mix, x, proj = case(n, 300, 600, seed=5 * n)
    if what == "tiny":
        mix, x = _scaled(mix, x, 2.0**-30)
    elif what == "huge":
        mix, x = _scaled(mix, x, 2.0**20)
    elif what == "far":
        mix, x = _scaled(mix, x, 1.0, 64.0)
    elif what == "one-point":   # tiles without extent
        x = np.repeat(mix["mean"][:3] + np.float32(0.01), 200, axis=0)
    elif what == "tile-1":
        tile = 1
    elif what == "wide-factors":
        mix, x, proj = case(n, 300, 600, seed=5 * n, sdiag=(0.1, 1000.0), soff=0.0)
    else:   # Gaussians of very different sizes side by side
        mix["factor"] = (mix["factor"] * np.float32(2.0) **
                         np.random.default_rng(n).integers(-12, 4, (300, 1))).astype(np.float32)
    _run(mix, x, proj, tile, tau)
