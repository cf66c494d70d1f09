"""tq_sketch_lowrank on tall narrow matrices: the left vectors are written by workgroups of their own, on fewer and on more rows
than one sweep of them covers (1024 workgroups of 256 rows); and the time of the calls that write them."""
import numpy as np
import pytest
import torch

from oracle.sketch_ref import sketch_lowrank
import paper_2605_09281_amd.binding as tq
from gpu_util import DEV
from test_gpu_sketch import TOL, run_gpu
from test_gpu_sketch_steps import TOL_NORM

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,cols,r,it", [(255, 4, 1, 0), (257, 8, 2, 1), (262144, 4, 2, 0), (300001, 4, 3, 1), (70001, 68, 3, 0)])
def test_tall_narrow(rows, cols, r, it):
    print(f"sketch {rows}x{cols} r={r} it={it}", flush=True)
    rng = np.random.default_rng(rows + cols)
    k = min(cols, 24)
    # the same construction, and the same bounds for the same reasons, as in test_gpu_sketch.py and test_gpu_sketch_steps.py
    W = (rng.standard_normal((rows, k)) * (0.7 ** np.arange(k))) @ rng.standard_normal((k, cols)) + 0.05 * rng.standard_normal((rows, cols))
    W = W.astype(np.float32)
    S = rng.standard_normal((r, cols)).astype(np.float32)
    U, sig, V, R = run_gpu(W, r, it, S)
    Uo, so, Vo, Ro = sketch_lowrank(W, r, it, S)
    for i in range(r):
        assert abs(sig[i] - so[i]) <= TOL * so[0], (i, sig[i], so[i])
        # 2-norms of unit vectors: the entries of U are too small for a bound on the largest one
        assert np.linalg.norm(U[i] - Uo[i]) <= TOL_NORM, i
        assert np.linalg.norm(V[i] - Vo[i]) <= TOL_NORM, i
    assert np.max(np.abs(R - Ro)) <= TOL * np.max(np.abs(W))


def test_writing_the_left_vectors_costs_less_than_the_passes():
    """One power iteration more is one pass more per rank.  Without any, a call is two block products, the left vectors and the
    residual: 580 us at 1000000 x 4, rank 4, against 1670 for four passes, 0.35 times; with the left vectors on one workgroup they
    alone took 3700, 2.2 times.  The bound lies in between."""
    r = 4
    W = torch.randn((1000000, 4), device=DEV)
    S = torch.randn((r, 4), device=DEV)
    ws = torch.empty(tq.lib().tq_sketch_workspace_size(1000000, 4), dtype=torch.uint8, device=DEV)
    t = {0: [], 1: []}
    for i in range(6):
        for it in (0, 1):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            tq.tq_sketch_lowrank(W, r, it, S, workspace=ws)
            b.record()
            b.synchronize()
            t[it].append(1000 * a.elapsed_time(b))
    t0, t1 = min(t[0]), min(t[1])
    print(f"sketch 1000000x4 rank {r}: {t0:.0f} us, with a power iteration {t1:.0f}", flush=True)
    assert t0 <= 2 * (t1 - t0)
