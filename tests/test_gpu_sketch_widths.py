"""tq_sketch_lowrank at the edges of its pass shapes: row lengths on either side of every switch of the workgroup width
(1024, 2048, 4096, 8192, 16384 and 32768 columns), row counts below and just past a whole number of row groups, and several
ranks."""
import numpy as np
import pytest

from oracle.sketch_ref import sketch_lowrank
from test_gpu_sketch import TOL, run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,cols,r,it", [(9, 1024, 3, 1), (8200, 1028, 3, 0), (4097, 2048, 4, 1), (1, 2052, 1, 0), (2051, 4096, 6, 1),
                                            (700, 4100, 6, 2), (513, 8192, 3, 1), (515, 8196, 7, 1), (300, 12672, 9, 2), (513, 16384, 4, 1),
                                            (257, 16388, 4, 2), (300, 32768, 3, 1), (40, 32772, 3, 1), (2, 4, 2, 2)])
def test_sketch_at_the_edges_of_the_pass_shapes(rows, cols, r, it):
    print(f"sketch {rows}x{cols} r={r} it={it}", flush=True)
    rng = np.random.default_rng(rows + cols)
    k = min(rows, cols, 24)
    # the same construction, and the same bound for the same reason, as in test_gpu_sketch.py
    W = (rng.standard_normal((rows, k)) * (0.7 ** np.arange(k))) @ rng.standard_normal((k, cols)) + 0.05 * rng.standard_normal((rows, cols))
    W = W.astype(np.float32)
    S = rng.standard_normal((r, cols)).astype(np.float32)
    U, sig, V, R = run_gpu(W, r, it, S)
    Uo, so, Vo, Ro = sketch_lowrank(W, min(r, rows), it, S[:min(r, rows)])
    for i in range(min(r, rows)):
        assert abs(sig[i] - so[i]) <= TOL * so[0], (i, sig[i], so[i])
        if so[i] > 1e-3 * so[0]:
            assert np.max(np.abs(U[i] - Uo[i])) <= TOL * 10, i
            assert np.max(np.abs(V[i] - Vo[i])) <= TOL * 10, i
    assert np.max(np.abs(R - Ro)) <= TOL * np.max(np.abs(W))
