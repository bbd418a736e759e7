"""The k-d order at the edges of its kernels, bit for bit against the CPU
re-implementation: subtree sizes (2,048 points; 1,024 where runs do not start
at multiples of 64 or there are more than 16 projections), nodes selected by
one workgroup (16,384), tiles that leave uneven runs, many tiles, and points whose
projections tie in whole runs, which the histogram's bins cannot separate."""

import numpy as np
import pytest

import oracle
from gpu_helpers import case, dev
from paper_2405_20067_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _check(mix, x, proj, tile, fields=("perm", "gperm", "tile_off", "cand")):
    from paper_2405_20067_amd import ngd
    k, n = mix["mean"].shape
    m = ngd.Mixture(n, k)
    m.update(*(dev(mix[f]) for f in ("mean", "factor", "weight", "colour")))
    p = ngd.default_params()
    p.tile, p.n_proj = tile, proj.shape[0]
    p.key_proj = min(p.key_proj, p.n_proj)
    xd = dev(x)
    c = ngd.Cull()
    for _ in range(2):   # a rebuild in the same buffers gives the same
        got = c.build(m, xd, proj, p).export()
        want = oracle.cull(mix["mean"], mix["factor"], x, proj, tau=p.tau, tile=tile,
                           key_proj=p.key_proj)
        for f in fields:
            np.testing.assert_array_equal(got[f], want[f], err_msg=f)


@pytest.mark.parametrize("q", [65, 128, 2047, 2048, 2049, 4097, 16384, 16385, 40001])
@pytest.mark.parametrize("tile", [64, 192, 256, 1024])
def test_sizes(torch_cuda, q, tile):
    # as many Gaussians as make their own order cross the same sizes
    mix, x, proj = case(3, max(65, q // 2), q, seed=q + tile)
    _check(mix, x, proj, tile)


@pytest.mark.parametrize("n_proj", [1, 5, 16, 17, 32])
def test_projection_counts(torch_cuda, n_proj):
    mix, x, _ = case(4, 2500, 9000, seed=n_proj)
    _check(mix, x, inputs.gen_projections(4, n_proj, seed=3), 256)


@pytest.mark.parametrize("q", [1500, 5000, 30000])
@pytest.mark.parametrize("what", ["same", "few", "steps", "one-off"])
def test_ties(torch_cuda, q, what):
    mix, x, proj = case(3, 3000, q, seed=q)
    rng = np.random.default_rng(q)
    if what == "same":          # every point the same
        x = np.repeat(x[:1], q, axis=0)
    elif what == "few":         # runs of equal points
        x = x[rng.integers(0, 7, q)]
    elif what == "steps":       # a coarse grid
        x = np.round(x * 4.0) / 4.0
    else:                       # one far point squeezes the rest into a bin
        x[q // 2] = 1e6
    mix["mean"][:] = x[rng.integers(0, q, 3000)]
    _check(mix, np.ascontiguousarray(x, dtype=np.float32), proj, 256)


@pytest.mark.parametrize("q", [4096, 4097, 16384, 16385, 65536, 65537])
def test_tile_counts(torch_cuda, q):
    # as many tiles as queries: the lists' offsets by one workgroup, in one
    # round, in several, and by the general scans
    mix, x, proj = case(2, 70, q, seed=q)
    _check(mix, x, proj, 1)


@pytest.mark.parametrize("n_proj", [3, 16, 20])
@pytest.mark.parametrize("q", [64 * 960, 64 * 1024 - 36])
def test_chunk_boxes(torch_cuda, q, n_proj):
    # 64 chunks against 15 and 16 groups of 64 tiles: the last size tested
    # without the chunks' boxes first and the first with them
    mix, x, _ = case(4, 4090, q, seed=n_proj)
    _check(mix, x, inputs.gen_projections(4, n_proj, seed=5), 64)


@pytest.mark.parametrize("q", [1500, 2048, 5000])
@pytest.mark.parametrize("far", [30.0, 3e3, 3e38])
def test_heavy_bins(torch_cuda, q, far):
    # bins of more than 64 points that a second histogram over the bin
    # separates wholly, in part, and not at all (the range is infinite)
    mix, x, proj = case(3, 3000, q, seed=q)
    x[q // 2] = far
    x[q // 3] = -far
    mix["mean"][:] = x[np.random.default_rng(q).integers(0, q, 3000)]
    # the orders alone: the lists of means whose projections overflow are not
    # the re-implementation's
    _check(mix, x, proj, 256, fields=("perm", "gperm"))


@pytest.mark.parametrize("q", [1 << 20, (1 << 20) + 1])
def test_scan_blocks(torch_cuda, q):
    # tiles of one query: as many counts as 256 blocks of a scan hold, the last
    # size whose blocks add up the sums before them, and one more
    mix, x, proj = case(1, 5, q, seed=1)
    _check(mix, x, proj, 1)
