"""n_chunks_unstaged: the strips of the enumeration that several waves share.
With one cell there is one group, and the number follows from the meshes'
sizes: runs of equal length over strips of 64 boxes."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,m,shape", [(8, 8, 0), (40, 16, 0), (40, 16, 1), (40, 16, 3), (96, 64, 0)])
def test_shared_strips(n, m, shape):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2109_14814_amd as ms
    A = synth.torus_mesh(n, m, synth.surface_coeffs(1))
    B = synth.torus_mesh(m, m, synth.surface_coeffs(2))
    lo = np.minimum(A.verts.min((0, 1)), B.verts.min((0, 1)))
    p = ms.make_params(lo, 1e-3, [1, 1, 1, 1])
    p.enum_shape = shape
    _, st, _ = ms.search(ms.Mesh.from_synth(A), ms.Mesh.from_synth(B), p, hits_cap=1 << 12)
    nA, nB = A.n_tris, B.n_tris
    assert st["n_groups"] == 1 and st["n_slots"] == nA * nB
    by_b, by_a = -(-nB // 64) * (nA + 16), -(-nA // 64) * (nB + 16)      # units: 16 for a strip's start
    units, strip = (by_b, nA + 16) if by_b <= by_a else (by_a, nB + 16)
    run = max(-(-units // 8192), {0: 32, 1: 64, 2: 32, 3: 16}[shape])    # 2048 blocks of four waves
    first = np.arange(0, units, strip)
    assert st["n_chunks_unstaged"] == np.count_nonzero(first // run != (first + strip - 1) // run)
