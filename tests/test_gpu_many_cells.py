"""Groups of many more distinct cells than the statistics' table holds (64): a
table of 2^8 hashed cells for grids of some cells to hundred thousands.  The
exact cells and slots against the oracle's, plain and in a batch."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("inv", [2.0, 10.0, 20.0, 40.0])
def test_cells_of_a_group(inv):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2109_14814_amd as ms
    A = synth.torus_mesh(24, 20, synth.surface_coeffs(5))
    B = synth.torus_mesh(24, 20, synth.surface_coeffs(5))
    B.verts += np.array([1e-3, 2e-3, -1e-3, 5e-4])
    V = np.concatenate([A.verts.reshape(-1, 4), B.verts.reshape(-1, 4)])
    lo, n = V.min(0) - 0.3 / inv, np.ceil((V.max(0) - V.min(0)) * inv).astype(np.int64) + 1
    ref, g = oracle.bruteforce(A, B), oracle.grid_search(A, B, lo, inv, n)
    ga, gb = ms.Mesh.from_synth(A), ms.Mesh.from_synth(B)
    p = ms.make_params(lo, inv, [int(k) for k in n], 0, table_log2=8)
    hits, st, _ = ms.search(ga, gb, p, hits_cap=1 << 14)
    print(f"  groups={st['n_groups']} cells={st['n_cells']} entries={st['n_entries']}", flush=True)
    assert np.array_equal((hits["triA"].astype(np.int64) << 32) | hits["triB"].astype(np.int64), ref.hit_pairs)
    assert st["n_cells"] == g.n_boxes and st["n_slots"] == g.n_slots
    b = ms.Batch([(ga, gb)] * 3, [p] * 3, hits_cap=1 << 16)
    b.run_checked(True)
    _, bst = b.results()
    assert bst["n_cells"] == 3 * g.n_boxes and bst["n_slots"] == 3 * g.n_slots
