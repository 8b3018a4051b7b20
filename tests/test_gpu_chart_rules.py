"""Chart points at the sizes where another kernel takes over: one query a block
and four (256 queries), four and sixteen on the matrix cores (1536, and where a
round of 4096 is full enough), and each order at which its step of orders
ends.  Reference and bars as for the other sizes of charts."""
import numpy as np
import pytest

from test_gpu_chart_sizes import LD, _partials, _reference, ms  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,order", [(32, 0), (32, 3), (33, 4), (2, 7), (32, 8), (1024, 0), (1024, 3), (64, 15), (64, 27),
                                     (64, 28)])
@pytest.mark.parametrize("nq", [256, 257, 1536, 1537, 4097])
def test_charts_on_both_sides(ms, N, order, nq):  # noqa: F811
    rng = np.random.default_rng(N + 31 * order + nq)
    spec = rng.standard_normal((order + 1, N, 4)) * 0.6 ** np.arange(order + 1)[:, None, None]
    theta, s = rng.uniform(-7, 7, nq), rng.uniform(-1, 1, nq)
    got = _partials(ms, spec, theta, s)
    n = N * (order + 1)
    for q in np.unique(np.r_[0, 15, 16, nq - 1, rng.integers(0, nq, 8)]):
        ref, size = _reference(spec, theta[q], s[q])
        for a, b, m in zip(got, ref, size):
            assert np.max(np.abs(a[q].astype(LD) - b)) <= 2.0 ** -50 * n ** 0.5 * m
    assert all(np.all(np.isfinite(a)) for a in got)
