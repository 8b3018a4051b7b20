"""The tangents on both sides of the batch size up to which a column runs on a
pair of lanes (5,461 hits) and between it and the states' (16,384)."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [5461, 5462, 8192, 10923])
def test_tangent_sizes(n):
    """The first and last hits of a batch against a batch of their own: the
    same to rounding (bar as for the two sides of the states' size)."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2109_14814_amd as ms
    x = np.random.default_rng(n).uniform(-1e-3, 1e-3, (n, 4))
    U, S = ms.patch_row(synth.patch_dirs(3, synth.UNSTABLE_BASE)), ms.patch_row(synth.patch_dirs(4, synth.STABLE_BASE))
    fwd, bwd = ms.MapParams(2.527e-5, 0.0094, 40, 1), ms.MapParams(2.527e-5, 0.0094, 40, -2)
    some = np.r_[0:33, n - 33:n]
    a = ms.refine_grad(x, U, S, fwd, bwd, ms.MS_REFINE_TANGENT)
    b = ms.refine_grad(x[some], U, S, fwd, bwd, ms.MS_REFINE_TANGENT)
    for k in ("f", "r", "J", "grad"):
        u, v = a[k].cpu().numpy()[some], b[k].cpu().numpy()
        assert np.max(np.abs(u - v)) <= 1e-11 * max(1.0, np.max(np.abs(v))), k
    xa, _, _, sa, _ = ms.refine_newton(x, U, S, fwd, bwd, max_trials=3)
    xb, _, _, sb, _ = ms.refine_newton(x[some], U, S, fwd, bwd, max_trials=3)
    assert np.array_equal(sa.cpu().numpy()[some], sb.cpu().numpy())
    assert np.max(np.abs(xa.cpu().numpy()[some] - xb.cpu().numpy())) <= 1e-9
