"""The pair enumeration at the sizes and grids where its strips, queues and
16-bit boxes can go wrong, against brute force: one group of nA x nB entries
around multiples of a wave, groups of many cells, worlds that the meshes
leave, and triangles wider than the offsets that an entry keeps."""
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


def _check(ms, A, B, lo, inv, n, **kw):
    ref = oracle.bruteforce(A, B)
    s = ms.Searcher(ms.Mesh.from_synth(A), ms.Mesh.from_synth(B),
                    ms.make_params(lo, inv, n, ms.MS_SEARCH_CANDIDATES, **kw), hits_cap=1 << 13, cand_cap=1 << 18)
    s.run()
    hits, st, cand = s.results()
    assert np.array_equal(np.sort(cand), ref.cand)
    assert np.array_equal((hits["triA"].astype(np.int64) << 32) | hits["triB"].astype(np.int64), ref.hit_pairs)
    for f in ("u", "v", "a", "b", "X", "thA", "sA", "thB", "sB", "margin"):
        assert len(hits) == 0 or np.max(np.abs(hits[f] - ref.hits[f])) <= 1e-10, f
    assert st["n_cand"] == len(ref.cand) and st["n_moller"] == ref.counts["moller_reject"]
    assert st["n_outside"] == ref.counts["outside"] and st["n_degenerate"] == ref.counts["degenerate"]
    return st, ref


@pytest.mark.parametrize("shape", [0, 1, 3])
@pytest.mark.parametrize("a,b", [((1, 1), (1, 1)), ((1, 1), (4, 8)), ((31, 1), (33, 1)), ((4, 8), (4, 8)),
                                 ((5, 13), (1, 1)), ((3, 11), (40, 40)), ((64, 8), (7, 3)), ((50, 21), (50, 20))])
def test_one_group(ms, a, b, shape):
    """All triangles in one cell: nA x nB slots, from 2 x 2 over 62 x 66, 64 x
    64 and 130 x 2 to crowded ones, most of them overlapping nothing."""
    A, B = synth.torus_mesh(*a, synth.surface_coeffs(3)), synth.torus_mesh(*b, synth.surface_coeffs(4))
    st, _ = _check(ms, A, B, [-3.0] * 4, 1.0 / 6.0, [1, 1, 1, 1], enum_shape=shape)
    assert st["n_groups"] == 1 and st["n_slots"] == st["n_group_slots"] == A.n_tris * B.n_tris


@pytest.mark.parametrize("table_log2", [8, 10])
def test_groups_of_many_cells(ms, table_log2):
    """Tables far too small: every group holds many cells, whose entries pair
    only within their cell, and more cells than the statistics' table has."""
    A, B = synth.plain_pair(40, 24, 2)
    lo, _, inv, n = oracle.default_grid([A, B], 0.5)
    st, _ = _check(ms, A, B, lo, inv, n, table_log2=table_log2)
    g = oracle.grid_search(A, B, lo, inv, n)
    assert st["n_cells"] == g.n_boxes and st["n_slots"] == g.n_slots < st["n_group_slots"]


@pytest.mark.parametrize("lo,inv,n", [((-0.3, -0.2, -0.2, -0.1), 4.0, (3, 2, 2, 2)), ((0.0, 0.0, 0.0, 0.0), 2.0, (1, 2, 3, 1)),
                                      ((5.0, -9.0, 0.0, 0.0), 1.0, (2, 2, 2, 2)), ((-2.0, -2.0, -2.0, -2.0), 40.0, (160,) * 4)])
def test_worlds_that_do_not_hold_the_meshes(ms, lo, inv, n):
    """Coordinates below and above the world take its first and last cells;
    in the finest grid the coarse mesh's triangles span more than 15 cells."""
    A, B = synth.torus_mesh(12, 6, synth.surface_coeffs(5)), synth.torus_mesh(48, 32, synth.surface_coeffs(6))
    for P, Q in ((A, B), (B, A)):
        st, _ = _check(ms, P, Q, list(lo), inv, list(n))
        g = oracle.grid_search(P, Q, np.array(lo), inv, np.array(n, np.int64))
        assert st["n_cells"] == g.n_boxes and st["n_slots"] == g.n_slots and st["n_entries_all"] == g.n_entries


def test_touching_boxes(ms):
    """Boxes that meet in a face or a point count as overlapping (closed
    intervals): a mesh against copies of itself, moved by whole quads."""
    th = np.arange(9) / 8.0
    A = synth.affine_mesh([0, 0, 0, 0], [1, 0, 0, 0], [0, 1, 0, 0], th, th)
    for dx, dy in ((0.0, 0.0), (1.0, 0.0), (0.5, 1.0), (1.0, 1.0)):
        B = synth.affine_mesh([dx, dy, 0, 0], [1, 0, 0.25, 0], [0, 1, 0, 0.25], th, th)
        _check(ms, A, B, [-0.25] * 4, 4.0, [12, 12, 4, 4])
        _check(ms, A, B, [-0.25] * 4, 1.0 / 3.0, [1, 1, 1, 1])


@pytest.mark.parametrize("table_log2", [0, 12])
@pytest.mark.parametrize("inv", [1.5, 9.0, 20.0, 30.0])
def test_ranges_of_many_blocks_and_regions(ms, inv, table_log2):
    """Triangles of one cell to more than 15 per axis: ranges inside a 2^4
    block, over several blocks and regions, tiles whose entries overflow the
    list of a block and ranges too wide for its words."""
    A, B = synth.torus_mesh(27, 20, synth.surface_coeffs(7)), synth.torus_mesh(16, 33, synth.surface_coeffs(8))
    V = np.concatenate([A.verts.reshape(-1, 4), B.verts.reshape(-1, 4)])
    lo, n = V.min(0) - 0.3 / inv, np.ceil((V.max(0) - V.min(0)) * inv).astype(np.int64) + 1
    st, _ = _check(ms, A, B, list(lo), inv, [int(k) for k in n], table_log2=table_log2)
    g = oracle.grid_search(A, B, lo, inv, n)
    assert st["n_cells"] == g.n_boxes and st["n_slots"] == g.n_slots and st["n_entries_all"] == g.n_entries
