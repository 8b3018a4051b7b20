"""The maps, the matrices and the refinement at the batch sizes where their
work is split differently: pairs of lanes for small batches (partial waves,
one block and several, the largest size), one lane per state above, several
launches when a round of blocks would be nearly empty.  Every size against
the oracle on the first, the last and some of its states."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

MU, ECC, STEPS = 2.527e-5, 0.0094, 600      # 600 steps: several chunks, and enough of them to be cut into launches


@pytest.fixture(scope="module")
def ms():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2109_14814_amd as ms
    ms.lib()
    return ms


def _sample(n):
    rng = np.random.default_rng(n)
    return np.unique(np.concatenate([[0, n - 1, n // 2], rng.integers(0, n, 13)]))


@pytest.mark.parametrize("n,periods", [(1, 1), (31, -1), (97, 1), (24576, 1), (24577, -1), (65536, 1), (65537, 1),
                                       (71680, -1), (131073, 1), (200001, 2)])
def test_maps(ms, n, periods):
    y = synth.random_states(n, n, spread=1e-3)
    z = synth.periapse_position_momentum(y, ECC)
    i = _sample(n)
    got = ms.propagate(y, MU, ECC, STEPS, periods).cpu().numpy()
    assert np.max(np.abs(got[i] - oracle.rk8_map(y[i], MU, ECC, STEPS, periods))) < 1e-10
    got = ms.pertbp_map(z, MU, ECC, STEPS, periods).cpu().numpy()
    assert np.max(np.abs(got[i] - oracle.pertbp_map(z[i], MU, ECC, STEPS, periods))) < 1e-10


@pytest.mark.parametrize("n", [1, 25, 6144, 6145, 16385, 32769, 65537, 70000])
def test_matrices(ms, n):
    z = synth.pm_random_states(n, n, ECC, spread=1e-3)
    i = _sample(n)
    out, M = (t.cpu().numpy() for t in ms.pertbp_map_stm(z, MU, ECC, STEPS, 1))
    ref, ref_M = oracle.pertbp_map(z[i], MU, ECC, STEPS, 1, stm=True)
    assert np.max(np.abs(out[i] - ref)) < 1e-10
    assert np.max(np.abs(M[i] - ref_M)) < 1e-10 * max(1.0, np.max(np.abs(ref_M)))
    # without the states there is nowhere to keep them between launches
    _, M1 = ms.pertbp_map_stm(z, MU, ECC, STEPS, 1, want_out=False)
    assert np.array_equal(M1.cpu().numpy(), M)


def test_in_place_over_several_launches(ms):
    import torch
    y = torch.tensor(synth.random_states(66000, 5, spread=1e-3), device="cuda")
    ref = ms.propagate(y, MU, ECC, STEPS, 1)
    assert torch.equal(ms.propagate(y, MU, ECC, STEPS, 1, out=y), ref)


def test_no_steps(ms):
    y = synth.random_states(66000, 6)
    for n in (40, 66000):
        assert np.array_equal(ms.pertbp_map(y[:n], MU, ECC, STEPS, 0).cpu().numpy(), y[:n])
        out, M = ms.pertbp_map_stm(y[:n], MU, ECC, STEPS, 0)
        assert np.array_equal(out.cpu().numpy(), y[:n])
        assert np.array_equal(M.cpu().numpy(), np.broadcast_to(np.eye(4), (n, 4, 4)))


@pytest.mark.parametrize("periods", [(3, -3), (3, -1), (0, -2)])
def test_gradient_for_every_checkpoint_interval(ms, periods):
    """The adjoint works on segments of its own: whatever the checkpoints'
    interval (above, below and at the segments' length) it gives the same
    bits, and the tangent's gradient to rounding."""
    steps, K = 130, 5
    rng = np.random.default_rng(1)
    x = rng.uniform(-1e-3, 1e-3, (K, 4))
    U, S = ms.patch_row(synth.patch_dirs(3, synth.UNSTABLE_BASE)), ms.patch_row(synth.patch_dirs(4, synth.STABLE_BASE))
    fwd, bwd = (ms.MapParams(MU, ECC, steps, p) for p in periods)
    ref = ms.refine_grad(x, U, S, fwd, bwd, ms.MS_REFINE_ADJOINT, 100)
    for ck in (1, 7, 99, 101, 250, 1000):
        got = ms.refine_grad(x, U, S, fwd, bwd, ms.MS_REFINE_ADJOINT, ck)
        for k in ("f", "r", "grad"):
            assert np.array_equal(got[k].cpu().numpy(), ref[k].cpu().numpy()), (ck, k)
    tan = ms.refine_grad(x, U, S, fwd, bwd, ms.MS_REFINE_TANGENT)["grad"].cpu().numpy()
    g = ref["grad"].cpu().numpy()
    assert np.max(np.abs(tan - g)) <= 1e-10 * max(1.0, np.max(np.abs(g)))


def test_refinement_on_both_sides_of_the_pair_size(ms):
    """16,385 hits run one lane per trajectory, 16,384 two: the same first
    hits to rounding, in every mode."""
    n, steps = 16385, 40
    rng = np.random.default_rng(2)
    x = rng.uniform(-1e-3, 1e-3, (n, 4))
    U, S = ms.patch_row(synth.patch_dirs(3, synth.UNSTABLE_BASE)), ms.patch_row(synth.patch_dirs(4, synth.STABLE_BASE))
    fwd, bwd = ms.MapParams(MU, ECC, steps, 1), ms.MapParams(MU, ECC, steps, -2)
    for mode, ck in ((ms.MS_REFINE_RESIDUAL, 100), (ms.MS_REFINE_TANGENT, 100), (ms.MS_REFINE_ADJOINT, 33)):
        a = ms.refine_grad(x, U, S, fwd, bwd, mode, ck)
        b = ms.refine_grad(x[:-1], U, S, fwd, bwd, mode, ck)
        for k in a:
            u, v = a[k][:-1].cpu().numpy(), b[k].cpu().numpy()
            assert np.max(np.abs(u - v)) <= 1e-11 * max(1.0, np.max(np.abs(v))), (mode, k)


def test_mismatch_gradient_is_of_the_call(ms):
    """The gradient that the forward call keeps is that of its inputs, also
    after they are overwritten; without gradients, and where the adjoint's
    interval is refused, the call is the residual alone."""
    import torch
    rng = np.random.default_rng(3)
    x = torch.tensor(rng.uniform(-1e-3, 1e-3, (6, 4)), device="cuda")
    e = torch.tensor(ECC, dtype=torch.float64, device="cuda")
    U, S = ms.patch_row(synth.patch_dirs(3, synth.UNSTABLE_BASE)), ms.patch_row(synth.patch_dirs(4, synth.STABLE_BASE))
    fwd, bwd = ms.MapParams(MU, ECC, 60, 1), ms.MapParams(MU, ECC, 60, -1)
    ref = ms.refine_grad(x, U, S, fwd, bwd, ms.MS_REFINE_ADJOINT)
    call = lambda p, ck=100: ms.mismatch_r(p, e, U, S, MU, 60, 1, -1, ck)  # noqa: E731
    p = x.clone().requires_grad_(True)
    r = call(p)
    with torch.no_grad():
        assert torch.equal(call(p), r)
        p.zero_()
    r.sum().backward()
    assert torch.equal(p.grad, ref["grad"][:, :4]) and torch.equal(r.detach(), ref["r"])
    q = x.clone().requires_grad_(True)
    r = call(q, 0)
    assert torch.equal(r.detach(), ref["r"])
    with pytest.raises(ms.MSearchError):
        r.sum().backward()
