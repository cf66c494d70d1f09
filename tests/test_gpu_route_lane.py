"""Routing inside the permutation's launch with a token's scores in one lane's registers: one expert to sixteen, one selection to all of them, one
token to a full wave, with a bias, with ties, infinities and the lowest finite value.  Bit for bit what tq_route gives."""
import numpy as np
import pytest
import torch

import paper_2605_09281_amd.binding as tq
from test_gpu_route_forward import both_ways, rcfg

pytestmark = pytest.mark.gpu

CASES = {f"{E}_experts_k{k}_{T}_tokens": (2901 + i, E, k, T)
         for i, (E, k, T) in enumerate(((1, 1, 64), (2, 2, 1), (7, 3, 63), (15, 15, 17), (16, 1, 64), (16, 16, 16), (16, 4, 64)))}


@pytest.mark.parametrize("with_bias", [False, True], ids=["plain", "bias"])
@pytest.mark.parametrize("name", list(CASES))
def test_routing_by_lane_equals_the_routing_kernel(name, with_bias):
    print(f"route lane {name} bias {with_bias}", flush=True)
    seed, E, k, T = CASES[name]
    rng = np.random.default_rng(seed)
    logits = np.round(rng.standard_normal((T, E)) * 2).astype(np.float32)       # many ties
    logits[rng.random((T, E)) < 0.1] = np.finfo(np.float32).min
    logits[1::3, E // 2] = -np.inf
    logits[:, 0] = np.where(np.isinf(logits).all(axis=1), 0, logits[:, 0])      # (a row of -inf alone has no weights)
    bias = (0.25 * np.arange(E, 0, -1)).astype(np.float32) if with_bias else None
    _, _, _, _, (idx, w, y), (idx2, w2, y2) = both_ways(rcfg(seed, E=E, k=k, T=T), tq.TQ_ACT_BF16, logits=logits, bias=bias)
    assert torch.equal(idx, idx2) and torch.equal(w.view(torch.int32), w2.view(torch.int32))
    assert torch.equal(y.view(torch.int16), y2.view(torch.int16))
