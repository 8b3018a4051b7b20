"""Tiles of 512 triangles with about 1024 entries (where a plain search
starts to count a tile's entries by groups), 2048 (a window of them) and
many times that, in few groups and in more than a tile's table holds, against
brute force and the oracle's grid: every entry has to get a place of its own."""
import copy

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ms():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2109_14814_amd as ms
    ms.lib()
    return ms


def _pair():
    """One tile of triangles and its copy beside it: nearly every cell of one
    is a cell of the other."""
    A = synth.torus_mesh(16, 16, synth.surface_coeffs(9))
    B = copy.deepcopy(A)
    B.verts += np.array([1e-3, 2e-3, -1e-3, 5e-4])
    return A, B


@pytest.mark.parametrize("table_log2", [8, 0])
@pytest.mark.parametrize("inv,entries", [(0.1, (512, 512)), (0.5, (700, 1024)), (1.0, (1025, 2048)), (1.5, (1025, 2048)),
                                         (2.0, (2049, 4096)), (4.0, (4097, 10000)), (8.0, (30000, 50000))])
def test_dense_tiles(ms, inv, entries, table_log2):
    A, B = _pair()
    V = np.concatenate([A.verts.reshape(-1, 4), B.verts.reshape(-1, 4)])
    lo, n = V.min(0) - 0.3 / inv, np.ceil((V.max(0) - V.min(0)) * inv).astype(np.int64) + 1
    ref, g = oracle.bruteforce(A, B), oracle.grid_search(A, B, lo, inv, n)
    assert entries[0] <= g.n_entries // 2 <= entries[1]
    s = ms.Searcher(ms.Mesh.from_synth(A), ms.Mesh.from_synth(B),
                    ms.make_params(lo, inv, [int(k) for k in n], ms.MS_SEARCH_CANDIDATES, table_log2=table_log2),
                    hits_cap=1 << 13, cand_cap=1 << 18)
    for _ in range(2):
        s.run()
        hits, st, cand = s.results()
        assert np.array_equal(np.sort(cand), ref.cand)
        assert np.array_equal((hits["triA"].astype(np.int64) << 32) | hits["triB"].astype(np.int64), ref.hit_pairs)
        assert st["n_cells"] == g.n_boxes and st["n_slots"] == g.n_slots and st["n_entries_all"] == g.n_entries
