"""Chart points where the blocks of four queries change their number of waves
(1024 queries, 4096 up to order 8, 8188 beyond) or give way to the matrix cores
and take over again, with steps of frequencies that the waves share unevenly,
on both sides of the order up to which a lane keeps three coefficients in flight.
Reference and bars as for the other sizes of charts."""
import numpy as np
import pytest

from test_gpu_chart_sizes import LD, _partials, _reference, ms  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,order", [(96, 2), (160, 3), (128, 8), (256, 2), (512, 8), (128, 9), (300, 28), (33, 28),
                                     (512, 0), (65, 1)])
@pytest.mark.parametrize("nq", [1024, 1025, 2049, 4096, 4097, 8188, 8189])
def test_charts_by_waves(ms, N, order, nq):  # noqa: F811
    rng = np.random.default_rng(N + 31 * order + nq)
    spec = rng.standard_normal((order + 1, N, 4)) * 0.6 ** np.arange(order + 1)[:, None, None]
    theta, s = rng.uniform(-7, 7, nq), rng.uniform(-1, 1, nq)
    got = _partials(ms, spec, theta, s)
    n = N * (order + 1)
    for q in np.unique(np.r_[0, 3, 4, nq - 1, rng.integers(0, nq, 6)]):
        ref, size = _reference(spec, theta[q], s[q])
        for a, b, m in zip(got, ref, size):
            assert np.max(np.abs(a[q].astype(LD) - b)) <= 2.0 ** -50 * n ** 0.5 * m
    assert all(np.all(np.isfinite(a)) for a in got)
