"""Triangles of more than 2^16 cells each, where a tile's total is summed in
64 bits beside its scan: with 32-bit and 64-bit cells, plain and in a batch,
with a workspace for all of them and without."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


def _sheet(n, seed):
    """n x 1 quads whose columns lie at opposite corners of the unit box in
    turn, so that every triangle's box spans it."""
    rng = np.random.default_rng(seed)
    th, s = np.linspace(0.0, 1.0, n + 1), np.array([0.0, 1.0])
    v = (np.arange(n + 1) % 2)[None, :, None] + rng.uniform(-0.05, 0.05, (2, n + 1, 4))
    return synth.Mesh(np.ascontiguousarray(v), th, s, False)


@pytest.mark.parametrize("cells64", [False, True])
def test_wide_triangles(cells64):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2109_14814_amd as ms
    A, B = _sheet(3, 1), _sheet(4, 2)
    lo, inv, n = np.full(4, -0.1), 18 / 1.2, np.full(4, 18, np.int64)
    ref, g = oracle.bruteforce(A, B), oracle.grid_search(A, B, lo, inv, n)
    assert g.n_entries > (A.n_tris + B.n_tris) << 16 and len(ref.cand) == A.n_tris * B.n_tris
    cells = [int(k) for k in n]
    if cells64:
        cells[0] = 1 << 31      # (an axis longer than the meshes: the same cells)
    ga, gb = ms.Mesh.from_synth(A), ms.Mesh.from_synth(B)
    p = ms.make_params(lo, inv, cells, ms.MS_SEARCH_CANDIDATES)
    s = ms.Searcher(ga, gb, p, hits_cap=1 << 10, cand_cap=1 << 10)
    s.run()
    hits, st, cand = s.results()
    assert np.array_equal(np.sort(cand), ref.cand)
    assert np.array_equal((hits["triA"].astype(np.int64) << 32) | hits["triB"].astype(np.int64), ref.hit_pairs)
    assert st["n_cells"] == g.n_boxes and st["n_slots"] == g.n_slots and st["n_entries_all"] == g.n_entries
    b = ms.Batch([(ga, gb), (ga, gb)], [p, p], hits_cap=1 << 10)
    b.run_checked(False)
    per_pair, bst = b.results()
    assert bst["n_slots"] == 2 * g.n_slots and bst["n_entries_all"] == 2 * g.n_entries
    for h in per_pair:
        assert np.array_equal((h["triA"].astype(np.int64) << 32) | h["triB"].astype(np.int64), ref.hit_pairs)
    # a workspace for a tenth of the entries: the overflow is seen, and grown out of
    small = ms.Searcher(ga, gb, p, hits_cap=1 << 10, cand_cap=1 << 10)
    small.ws_bytes -= int(0.9 * 66 * g.n_entries)
    small.run_async()
    with pytest.raises(ms.MSearchError):
        small.check_overflow()
    assert small.stats.view(torch.int64).cpu().tolist()[0] > 0.5 * g.n_entries
    small.run()
    assert small.results()[1]["n_hits"] == len(ref.hits)
