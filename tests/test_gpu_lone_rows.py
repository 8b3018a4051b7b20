"""theta_spectrum on both sides of the numbers of rows at which rows of 256 to
1024 samples have a workgroup of their own (up to 1024 rows, and from 2^22
samples on; 256 samples always), in place too.  The bar of the rows that share
workgroups."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,n_rows", [(256, 1024), (256, 1537), (256, 16385), (512, 1024), (512, 1025), (512, 8191),
                                      (512, 8192), (1024, 1024), (1024, 1025), (1024, 4095), (1024, 4097)])
def test_spectrum_of_lone_and_shared_rows(N, n_rows):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2109_14814_amd as ms
    rng = np.random.default_rng(N + n_rows)
    rows = rng.standard_normal((n_rows, N, 4))
    some = np.unique(np.r_[0:40, 1020:1026, n_rows - 9:n_rows])
    some = some[some < n_rows]
    z = np.fft.fft(rows[some].reshape(len(some), N, 2, 2) @ np.array([1.0, 1j]), axis=1) / N
    ref = np.stack([z.real, z.imag], -1).reshape(len(some), N, 4)
    x = torch.from_numpy(rows).cuda()
    got = ms.theta_spectrum(x)
    assert np.max(np.abs(got.cpu().numpy()[some] - ref)) < 1e-13 * np.abs(rows).max() * np.log2(N)
    # every row against the same row in a call of few
    for r in (0, n_rows // 2, n_rows - 8):
        few = ms.theta_spectrum(x[r:r + 8].clone())
        assert torch.max(torch.abs(few - got[r:r + 8])).item() < 2e-13 * np.abs(rows).max() * np.log2(N)
    ms.theta_spectrum(x, out=x)
    assert torch.equal(x, got)
