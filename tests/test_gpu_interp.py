"""theta_interp at the row lengths and row orders where its tables, its tiles
of queries and its grouping by rows can go wrong, against the oracle's
trigonometric interpolation.  Bar: 1e-11 x max|a|, as for the other lengths."""
import numpy as np
import pytest

from oracle import spectral

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ms():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2109_14814_amd as ms
    ms.lib()
    return ms


def _check(ms, rows, at, theta, rng, n=250):
    import torch
    got = ms.theta_interp(rows, at, theta).cpu().numpy()
    rows = rows.cpu().numpy() if torch.is_tensor(rows) else rows
    good = (at >= 0) & (at < len(rows)) & np.isfinite(theta)
    assert np.all(np.isnan(got[~good])) and np.all(np.isfinite(got[good]))
    idx = np.flatnonzero(good & (np.abs(theta) < 1e4))
    idx = np.unique(np.concatenate([idx[:20], idx[-20:], rng.choice(idx, min(n, len(idx)))]))
    ref = np.stack([spectral.interpolate(rows[at[q]], theta[q]) for q in idx])
    assert np.max(np.abs(got[idx] - ref)) < 1e-11 * np.abs(rows).max()


def _theta(n, N, rng):
    th = rng.uniform(-10, 10, n)
    k = rng.integers(0, n, max(1, n // 50))
    th[k] = 2 * np.pi * rng.integers(-2 * N, 2 * N, len(k)) / N                      # at samples
    th[rng.integers(0, n, 2)] = 2 * np.pi * 3 / N * (1 + 1e-15)                      # next to one
    return th


@pytest.mark.parametrize("N", [63, 64, 65, 127, 128, 129, 255, 256, 257, 300, 511, 512, 513, 1021, 2047, 2048, 2049])
@pytest.mark.parametrize("nq", [3, 700, 17000])
def test_row_lengths(ms, N, nq):
    """Lengths around the steps of 64 and 256 samples, even and odd; one query
    per wave, and several of a row."""
    rng = np.random.default_rng(N + nq)
    rows = rng.standard_normal((9, N, 4))
    _check(ms, rows, rng.integers(0, 9, nq), _theta(nq, N, rng), rng)


@pytest.mark.parametrize("N,n_rows", [(2048, 160), (2047, 160), (320, 1100), (64, 20000)])
@pytest.mark.parametrize("order", ["random", "sorted", "one", "skewed", "few", "two_slices"])
def test_grouped_by_rows(ms, N, n_rows, order):
    """Rows of more than 8 MB with at least two queries each, in any order:
    rows with more queries than a block takes, rows that do not exist, angles
    too large to mean anything among the others, bins of several rows."""
    import torch
    rng = np.random.default_rng(n_rows)
    nq = 70001 if order == "two_slices" else max(4096, 2 * n_rows) + 77
    at = rng.integers(0, n_rows, nq)
    if order == "sorted":
        at.sort()
    elif order == "one":
        at[:] = n_rows - 1
    elif order == "skewed":
        at[rng.uniform(size=nq) < 0.5] = 11
    elif order == "few":
        at = rng.integers(0, 3, nq) * 50
    theta = _theta(nq, N, rng)
    at[rng.integers(0, nq, 9)] = rng.choice([-1, n_rows, 1 << 40, -(1 << 40)], 9)
    theta[rng.integers(0, nq, 9)] = np.nan
    theta[rng.integers(0, nq, 9)] = 1e18
    rows = torch.from_numpy(rng.standard_normal((n_rows, N, 4))).cuda()
    _check(ms, rows, at, theta, rng)


@pytest.mark.parametrize("N", [2, 4, 8, 16, 64, 512, 1024, 2048])
@pytest.mark.parametrize("n_rows", [1, 7, 301])
def test_rows_per_workgroup(ms, N, n_rows):
    """theta_shift and theta_spectrum where a workgroup takes several rows and
    the last one not all of them; shifts so large that the phases' table does
    not reach.  Bars: 1e-13 N^order x max|a|, the spectrum 1e-13 x log2 N."""
    rng = np.random.default_rng(N + n_rows)
    rows = rng.standard_normal((n_rows, N, 4))
    rho = rng.uniform(-4, 4, n_rows)
    rho[::5] *= 1e6
    for order in (0, 1, 2):
        got = ms.theta_shift(rows, rho, order).cpu().numpy()
        ref = spectral.shift_derivative(rows, rho, order)
        assert np.max(np.abs(got - ref)) < 1e-13 * N ** order * max(1.0, np.abs(rows).max()) * max(1.0, np.log2(N))
    z = np.fft.fft(rows.reshape(n_rows, N, 2, 2) @ np.array([1.0, 1j]), axis=1) / N
    ref = np.stack([z.real, z.imag], -1).reshape(n_rows, N, 4)
    assert np.max(np.abs(ms.theta_spectrum(rows).cpu().numpy() - ref)) < 1e-13 * np.abs(rows).max() * max(1.0, np.log2(N))
