"""A chart with an infinite coefficient at the cosine mode N / 2: what it is
part of is infinite, everything else as if it were not there.  One query per
block, four, and sixteen on the matrix cores (which leave such queries to the
first form)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nq", [5, 300, 2311])
@pytest.mark.parametrize("N,order", [(64, 3), (512, 9)])
def test_infinite_cosine_mode(N, order, nq):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2109_14814_amd as ms
    rng = np.random.default_rng(N + nq)
    chart = ms.FourierTaylor(rng.standard_normal((order + 1, N, 4)) * 0.5 ** np.arange(order + 1)[:, None, None])
    th, s = rng.uniform(0, 6, nq), rng.uniform(-1, 1, nq)
    chart.spec[0, N // 2, 1] = 0.0
    w0, dth0, ds0 = (t.cpu().numpy() for t in chart.partials(th, s))
    chart.spec[0, N // 2, 1] = float("inf")
    w, dth, ds = (t.cpu().numpy() for t in chart.partials(th, s))
    cos = np.cos(N // 2 * th)
    sure = np.abs(cos) > 1e-9
    assert np.array_equal(w[sure, 1], np.copysign(np.inf, cos[sure]))
    scale = 1e-12 * N                                       # (N^2 terms of order 1 in dth, each to an ulp or two)
    assert np.max(np.abs(np.delete(w, 1, 1) - np.delete(w0, 1, 1))) < scale
    assert np.max(np.abs(dth - dth0)) < scale * N and np.max(np.abs(ds - ds0)) < scale
