"""theta_shift and theta_spectrum on both sides of the number of rows up to
which a row has a workgroup of its own (768, or twice that), in place too, with shifts beyond
the phases' table.  Bars as for the rows per workgroup."""
import numpy as np
import pytest

from oracle import spectral

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [2, 4, 8, 16, 32, 64, 128, 256, 512, 1024])
@pytest.mark.parametrize("n_rows", [2, 768, 769, 1537])
def test_few_and_many_rows(N, n_rows):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2109_14814_amd as ms
    rng = np.random.default_rng(N + n_rows)
    rows = rng.standard_normal((n_rows, N, 4))
    rho = rng.uniform(-4, 4, n_rows)
    rho[1::5] *= 1e6
    some = np.unique(np.r_[0:min(n_rows, 40), n_rows - 1])
    x = torch.from_numpy(rows).cuda()
    for order in (0, 1, 2):
        got = ms.theta_shift(x, rho, order)
        ref = spectral.shift_derivative(rows[some], rho[some], order)
        bar = 1e-13 * N ** order * max(1.0, np.abs(rows).max()) * max(1.0, np.log2(N))
        assert np.max(np.abs(got.cpu().numpy()[some] - ref)) < bar
        y = x.clone()
        ms.theta_shift(y, rho, order, out=y)
        assert torch.equal(y, got)
    one = ms.theta_shift(x[:1].clone(), 0.3, 1).cpu().numpy()
    assert np.max(np.abs(ms.theta_shift(x, 0.3, 1).cpu().numpy()[:1] - one)) < 1e-13 * N * 6 * max(1.0, np.log2(N))
    z = np.fft.fft(rows.reshape(n_rows, N, 2, 2) @ np.array([1.0, 1j]), axis=1) / N
    ref = np.stack([z.real, z.imag], -1).reshape(n_rows, N, 4)
    got = ms.theta_spectrum(x)
    assert np.max(np.abs(got.cpu().numpy() - ref)) < 1e-13 * np.abs(rows).max() * max(1.0, np.log2(N))
    ms.theta_spectrum(x, out=x)
    assert torch.equal(x, got)
