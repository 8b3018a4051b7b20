"""What a Searcher holds after run() had to grow its records: one allocation
for counters and records, and `stats` still the tensor that a caller may hold."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hits_cap", [0, 1, 50])
def test_grown_searcher(hits_cap):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2109_14814_amd as ms
    rng = np.random.default_rng(5)
    A, B = (synth.torus_mesh(12, 12, synth.surface_coeffs(k)) for k in (1, 2))
    A.verts[...] = rng.uniform(-1, 1, A.verts.shape)
    B.verts[...] = rng.uniform(-1, 1, B.verts.shape)
    ref = oracle.bruteforce(A, B)
    assert len(ref.hits) > 128
    lo, _, inv, cells = oracle.default_grid([A, B], 2.0)
    s = ms.Searcher(ms.Mesh.from_synth(A), ms.Mesh.from_synth(B), ms.make_params(lo, inv, cells), hits_cap=hits_cap)
    held = s.stats
    s.run()
    assert s.hits_cap >= len(ref.hits) and s.stats is held
    assert held.untyped_storage().data_ptr() == s.hits.untyped_storage().data_ptr()
    assert s.hits.data_ptr() == held.data_ptr() + 128 and s.hits.numel() == s.hits_cap * ms.HIT_DTYPE.itemsize
    for _ in range(2):
        hits, st, _ = s.results()
        assert st["n_hits"] == len(ref.hits) and held.view(torch.int64)[8].item() == len(ref.hits)
        assert np.array_equal((hits["triA"].astype(np.int64) << 32) | hits["triB"].astype(np.int64), ref.hit_pairs)
        s.run()
