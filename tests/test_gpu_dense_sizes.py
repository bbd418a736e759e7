"""The unculled forward and backward at the edges of their launch rules (one,
two and four queries a lane, split or whole mixtures, 4 / 8 / 16 waves a
Gaussian), against the float64 oracle at the float32 bar of the parity tests
(1e-4 of the output's scale)."""

import pytest

import oracle
from gpu_helpers import case, dev, host, normwise
from paper_2405_20067_amd import inputs

pytestmark = pytest.mark.gpu
TOL_FP32 = 1e-4


def _mixture(mix):
    from paper_2405_20067_amd import ngd
    m = ngd.Mixture(mix["mean"].shape[1], mix["mean"].shape[0])
    m.update(dev(mix["mean"]), dev(mix["factor"]), dev(mix["weight"]), dev(mix["colour"]))
    return m


# q below / at / above each rule's edge and its last partial wave; k below the
# number of waves that split it, one more than a multiple of it, odd
@pytest.mark.parametrize("n,k,q", [(1, 3, 1), (4, 5, 63), (10, 17, 65), (12, 31, 4097),
                                   (4, 33, 32768), (11, 16, 32770), (6, 40, 65535),
                                   (3, 1, 65537), (5, 65, 262143), (2, 9, 262401),
                                   (7, 6, (1 << 20) - 1), (4, 7, (1 << 20) + 769)])
def test_dense_forward_at_the_edges(n, k, q):
    from paper_2405_20067_amd import ngd
    mix, x, _ = case(n, k, q, seed=k + n)
    f = host(ngd.eval_mixture(_mixture(mix), None, dev(x)))
    want = oracle.eval_mixture(mix["mean"], mix["factor"], mix["weight"], mix["colour"], x)
    assert normwise(f, want) <= TOL_FP32


@pytest.mark.parametrize("n,k,q", [(1, 2, 1), (4, 3, 64), (9, 5, 1023), (10, 7, 1025),
                                   (11, 9, 700), (12, 4, 2049), (3, 4095, 130), (10, 4097, 70)])
def test_dense_backward_at_the_edges(n, k, q):
    from paper_2405_20067_amd import ngd
    mix, x, _ = case(n, k, q, seed=k + n)
    g = inputs.gen_grad_out(q, seed=n)
    got = [host(t) for t in ngd.eval_backward(_mixture(mix), None, dev(x), dev(g))]
    want = oracle.grad(mix["mean"], mix["factor"], mix["weight"], mix["colour"], x, g)
    for name, a, b in zip(("mean", "factor", "weight", "colour"), got, want):
        if abs(b).max() < 1e-30:   # G itself is below float32's range (n = 1, one far query)
            assert abs(a).max() < 1e-30, name
            continue
        assert normwise(a, b) <= TOL_FP32, name
