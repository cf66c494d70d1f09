"""tq_route with more than 16 selections (a wave per token): every number of scores per lane, at the edges of each, against the
oracle; and no more scores per lane than the experts need, seen in the time."""
import numpy as np
import pytest
import torch

import oracle
import paper_2605_09281_amd.binding as tq

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("E", [17, 63, 64, 65, 128, 129, 256, 257])
@pytest.mark.parametrize("T", [1, 131])
def test_many_selections(E, T):
    print(f"route E={E} T={T}", flush=True)
    rng = np.random.default_rng(77 * E + T)
    for k in sorted({17, min(E, 33), min(E, 64)}):
        logits = np.round(rng.standard_normal((T, E)) * 4).astype(np.float32) / 4      # ties
        bias = rng.standard_normal(E).astype(np.float32) if k == 17 else None
        idx, w = tq.tq_route(torch.from_numpy(logits).to(DEV), None if bias is None else torch.from_numpy(bias).to(DEV), k)
        torch.cuda.synchronize()
        ridx, rw = oracle.route(logits, bias, k)
        assert np.array_equal(idx.cpu().numpy(), ridx)
        assert np.max(np.abs(w.cpu().numpy() - rw)) <= 1e-6


def test_scores_per_lane_follow_the_experts():
    """64 selections of 64 experts (one score per lane) take less time than of 256 (four): 0.87 of it, and 1.00 where both run
    with room for four.  Timed in turn, the bound lies in the middle."""
    k, T = 64, 65536
    args = {E: (torch.randn((T, E), device=DEV), torch.empty((T, k), dtype=torch.int32, device=DEV), torch.empty((T, k), device=DEV))
            for E in (64, 256)}
    ratios = []
    for i in range(11):
        t = {}
        for E, (logits, idx, w) in args.items():
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            tq.tq_route(logits, None, k, idx, w)
            b.record()
            b.synchronize()
            t[E] = a.elapsed_time(b)
        ratios.append(t[64] / t[256])
    r = float(np.median(ratios))
    print(f"route of 64 against 256 experts, 64 selections: {r:.3f}", flush=True)
    assert r <= 0.93
