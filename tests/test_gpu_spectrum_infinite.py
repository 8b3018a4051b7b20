"""Spectra of rows with a sample that is no number or infinite in one
coordinate: the sums that it is no part of stay numbers, as in a transform that
leaves out its factors of 1."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [4, 16, 64, 128, 256, 512, 2048])
@pytest.mark.parametrize("n_rows", [3, 1600])
@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_one_bad_coordinate(N, n_rows, bad):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2109_14814_amd as ms
    rng = np.random.default_rng(N)
    x = rng.standard_normal((n_rows, N, 4))
    x[1, 5 % N, 1] = bad
    x[2, N - 1, 2] = bad
    z = ms.theta_spectrum(x).cpu().numpy()
    mean = x.mean(1)
    for row, comp in ((1, 1), (2, 2)):
        rest = [c for c in range(4) if c != comp]
        assert np.max(np.abs(z[row, 0, rest] - mean[row, rest])) < 1e-13 and not np.isfinite(z[row, 0, comp])
        other = [c for c in range(4) if c // 2 != comp // 2]
        assert np.all(np.isfinite(z[row][:, other]))
    assert np.all(np.isfinite(z[0])) and np.all(np.isfinite(z[3:]))
