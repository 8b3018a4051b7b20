"""Points and partials of a local chart at the orders, lengths and numbers of
queries where the kernels change or leave a remainder, against a plain sum in
longer arithmetic.  Bars: the terms' magnitudes are summed too, and a sum of
n terms may be off by n^(1/2) 2^-50 of that (the theta partial likewise);
nothing is compared where Horner's rule itself gives no number."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
LD = np.longdouble


@pytest.fixture(scope="module")
def ms():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2109_14814_amd as ms
    ms.lib()
    return ms


def _partials(ms, spec, theta, s):
    import torch
    d = [torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (spec, theta, s)]
    o = [torch.full((len(theta), 4), 7.0, dtype=torch.float64, device="cuda") for _ in range(3)]
    rc = ms.lib().ft_partials(d[0].data_ptr(), spec.shape[1], spec.shape[0] - 1, d[1].data_ptr(), d[2].data_ptr(),
                              len(theta), 0.0, 1.0, None, o[0].data_ptr(), o[1].data_ptr(), o[2].data_ptr(), None,
                              ctypes.c_void_p(0))
    assert rc == 0
    torch.cuda.synchronize()
    return [x.cpu().numpy() for x in o]


def _reference(spec, theta, s):
    n, P = spec.shape[1], spec.shape[0] - 1
    j = np.arange(n)
    j = np.where(2 * j > n, j - n, j).astype(np.float64)
    ph = (theta * j).astype(LD)                                # the product in 64 bits
    c, sn = np.cos(ph), np.where(2 * j == n, 0, np.sin(ph))
    jd = np.where(2 * j == n, 0, j).astype(LD)[:, None]
    pw = LD(s) ** np.arange(P + 1)
    dp = np.concatenate([[LD(0)], np.arange(1, P + 1) * pw[:-1]])

    def turn(v, c, sn):
        return np.stack([v[:, 0] * c - v[:, 1] * sn, v[:, 0] * sn + v[:, 1] * c,
                         v[:, 2] * c - v[:, 3] * sn, v[:, 2] * sn + v[:, 3] * c], 1)

    def sums(spec, pw, dp, c, sn, jd, sign):
        r = turn(np.tensordot(pw, spec, 1), c, sn)
        t = np.stack([sign * jd[:, 0] * r[:, 1], jd[:, 0] * r[:, 0], sign * jd[:, 0] * r[:, 3], jd[:, 0] * r[:, 2]], 1)
        return r.sum(0), t.sum(0), turn(np.tensordot(dp, spec, 1), c, sn).sum(0)

    ref = sums(spec.astype(LD), pw, dp, c, sn, jd, -1)
    size = sums(np.abs(spec).astype(LD), np.abs(pw), np.abs(dp), np.ones_like(c), -np.ones_like(c), np.abs(jd), 1)
    return ref, [np.abs(x).max() for x in size]


@pytest.mark.parametrize("nq", [1, 255, 256, 257, 2303, 2304, 2319])
@pytest.mark.parametrize("n,P", [(1, 0), (2, 1), (15, 3), (16, 4), (17, 7), (33, 8), (64, 15), (100, 16), (257, 27),
                                 (130, 28), (512, 5), (512, 25)])
def test_orders_and_lengths(ms, n, P, nq):
    rng = np.random.default_rng(100 * P + n)
    spec = rng.standard_normal((P + 1, n, 4))
    theta, s = rng.uniform(-10, 10, nq), rng.uniform(-1.1, 1.1, nq)
    s[0] = 0.0
    theta[-1] = 2e5                                            # phases beyond the table's range
    got = _partials(ms, spec, theta, s)
    for q in sorted({0, 1 % nq, nq // 2, max(0, nq - 17), max(0, nq - 2), nq - 1}):
        ref, size = _reference(spec, theta[q], s[q])
        for g, r, m in zip(got, ref, size):
            assert np.max(np.abs(g[q] - r)) <= np.sqrt(n * (P + 1.0)) * 2.0 ** -50 * m


@pytest.mark.parametrize("nq", [7, 300, 2400])
def test_numbers_that_are_none(ms, nq):
    """What is no number stays with its query, and where Horner's rule gives a
    number, a power or a product that is none does not spoil it."""
    rng = np.random.default_rng(nq)
    spec = rng.standard_normal((21, 64, 4))
    spec[3:] = 0.0
    theta, s = rng.uniform(-3, 3, nq), rng.uniform(-0.9, 0.9, nq)
    s[2], s[4], theta[5] = 1e20, np.nan, np.inf                # (1e20)^16 is no number
    got = _partials(ms, spec, theta, s)
    good = np.ones(nq, bool)
    good[[4, 5]] = False
    for g in got:
        assert np.all(np.isfinite(g[good])) and np.all(np.isnan(g[~good]))
    for q in (0, 2, 3, nq - 1):
        ref, size = _reference(spec[:3], theta[q], s[q])
        for g, r, m in zip(got, ref, size):
            assert np.max(np.abs(g[q] - r)) <= 14.0 * 2.0 ** -50 * m
    spec[0, 5, 1] = np.nan                                     # the s-partial never meets it
    w, dth, ds = _partials(ms, spec, theta, s)
    assert np.all(np.isnan(w[good][:, :2])) and np.all(np.isfinite(ds[good])) and np.all(np.isfinite(w[good][:, 2:]))
    assert np.array_equal(ds[good], got[2][good]) or np.max(np.abs(ds[good] / got[2][good] - 1)) < 1e-10
