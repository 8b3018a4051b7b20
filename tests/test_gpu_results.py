"""Searcher.results() around the records that it reads along with the
counters: none, fewer, more, and buffers that run() had to grow, each against
the device buffers themselves and the oracle's hit pairs."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hits_cap", [0, 1, 100, 128, 1 << 13])
@pytest.mark.parametrize("n,apart", [(3, 9.0), (2, 0.0), (5, 0.0), (12, 0.0)])
def test_results_match_the_buffers(n, apart, hits_cap):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2109_14814_amd as ms
    rng = np.random.default_rng(5)
    A, B = (synth.torus_mesh(n, n, synth.surface_coeffs(k)) for k in (1, 2))
    A.verts[...] = rng.uniform(-1, 1, A.verts.shape)
    B.verts[...] = rng.uniform(-1, 1, B.verts.shape) + apart
    ref = oracle.bruteforce(A, B)
    lo, _, inv, cells = oracle.default_grid([A, B], 2.0)
    s = ms.Searcher(ms.Mesh.from_synth(A), ms.Mesh.from_synth(B), ms.make_params(lo, inv, cells), hits_cap=hits_cap)
    for _ in range(2):
        s.run()
        hits, st, cand = s.results()
        assert cand is None and st["n_hits"] == len(hits) == len(ref.hits)
        assert np.array_equal((hits["triA"].astype(np.int64) << 32) | hits["triB"].astype(np.int64), ref.hit_pairs)
        size = ms.HIT_DTYPE.itemsize
        assert hits.tobytes() == s.hits[:len(hits) * size].cpu().numpy().tobytes()
        counters = s.stats.view(torch.int64).cpu().tolist()
        assert [st[k] for k in ms.STATS_FIELDS] == counters[:len(ms.STATS_FIELDS)]
