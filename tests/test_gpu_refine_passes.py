"""The passes of a Newton refinement that has nothing left to do: all of them
are queued in advance, and one without a running hit has to end at once."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [1, 100])
def test_passes_without_a_running_hit(K):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2109_14814_amd as ms
    x = np.random.default_rng(K).uniform(-1e-3, 1e-3, (K, 4))
    U, S = ms.patch_row(synth.patch_dirs(3, synth.UNSTABLE_BASE)), ms.patch_row(synth.patch_dirs(4, synth.STABLE_BASE))
    fwd, bwd = (ms.MapParams(2.527e-5, 0.0094, 4000, p) for p in (1, -1))
    run = lambda: ms.refine_newton(x, U, S, fwd, bwd, max_trials=20, tol=1e9)  # noqa: E731
    run()
    ms.profile_enable()
    try:
        xo, f, r, status, trials = run()
        times = [t for name, t in ms.profile_read() if name == "k_ref_tangent"]
    finally:
        ms.profile_enable(False)
    assert torch.all(status == 0) and torch.all(trials == 0) and np.array_equal(xo.cpu().numpy(), x)
    # every hit is done after the first pass (milliseconds); what the others
    # take is a launch, not 4,000 steps' barriers and loads (a 65th of the first)
    assert len(times) == 21 and sorted(times[1:])[10] < times[0] / 300
