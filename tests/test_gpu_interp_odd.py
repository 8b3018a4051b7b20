"""theta_interp at odd row lengths on both sides of the number of queries (4096)
and the length (512) up to which they are interpolated without the row length's
table, and where blocks of few queries hold the longest tables.  Bar: 1e-11 x
max|a|, as for the other lengths."""
import numpy as np
import pytest

from test_gpu_interp import _check, _theta, ms  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [319, 321, 511, 513, 1023, 2047])
@pytest.mark.parametrize("nq", [2047, 4096, 4097])
def test_odd_lengths(ms, N, nq):  # noqa: F811
    rng = np.random.default_rng(N + nq)
    n_rows = 600
    rows = rng.standard_normal((n_rows, N, 4))
    at = rng.integers(0, n_rows, nq)
    at[5], at[-1] = -1, n_rows
    theta = _theta(nq, N, rng)
    theta[7] = np.nan
    _check(ms, rows, at, theta, rng, n=120)
