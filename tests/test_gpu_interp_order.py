"""A query's interpolated value depends on its row and theta alone: not on the
other queries of the call, their order, or the order in which they are taken
(bit for bit), wherever the row length's table is used."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [256, 300, 511, 1024, 2047, 2048])
@pytest.mark.parametrize("n_rows", [3, 700])
def test_same_bits_in_any_company(N, n_rows):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2109_14814_amd as ms
    rng = np.random.default_rng(N + n_rows)
    rows = torch.from_numpy(rng.standard_normal((n_rows, N, 4))).cuda()
    nq = 20000
    at = rng.integers(0, n_rows, nq)
    theta = rng.uniform(-10, 10, nq)
    theta[::97] = 1e18                                         # (offsets of more than a step)
    theta[::89] = 2 * np.pi * rng.integers(0, N, len(theta[::89])) / N
    at, theta = torch.from_numpy(at).cuda(), torch.from_numpy(theta).cuda()
    first = ms.theta_interp(rows, at, theta)
    bits = lambda t: t.view(torch.int64)  # noqa: E731
    for _ in range(3):
        assert torch.equal(bits(ms.theta_interp(rows, at, theta)), bits(first))
    p = torch.from_numpy(rng.permutation(nq)).cuda()
    assert torch.equal(bits(ms.theta_interp(rows, at[p], theta[p])), bits(first[p]))
    by_row = torch.argsort(at)
    assert torch.equal(bits(ms.theta_interp(rows, at[by_row], theta[by_row])), bits(first[by_row]))
    for few in (5000, 16383):
        assert torch.equal(bits(ms.theta_interp(rows, at[:few], theta[:few])), bits(first[:few]))
