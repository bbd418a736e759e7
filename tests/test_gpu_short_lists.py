"""The culled forward on both sides of the list length up to which every candidate
is evaluated without the filter (12 an item, 64 up to three dimensions, any in
one): the same bounds as the filter's own test."""

import pytest

from gpu_helpers import case
from test_gpu_filter import _run, torch_cuda  # noqa: F401 (the fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,k", [(1, 12), (1, 700), (2, 64), (2, 65), (3, 64), (3, 65), (4, 12),
                                 (4, 13), (7, 12), (7, 13), (11, 12), (11, 13)])
@pytest.mark.parametrize("tile", [1, 100, 512])
def test_list_lengths(torch_cuda, n, k, tile):  # noqa: F811
    # a threshold that leaves every Gaussian a candidate of every tile
    mix, x, proj = case(n, k, 150, seed=n + k)
    _run(mix, x, proj, tile, 1e-30)
