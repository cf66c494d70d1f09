"""Routing with a row of 16 lanes per token (up to 256 experts and 16 selections) and the permutation with a workgroup per
1024 assignments, at the edges of their ranges: bit-exact indices against the oracle, weights within a few fp32 ulps."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

import oracle  # noqa: E402
import paper_2605_09281_amd.binding as tq  # noqa: E402

DEV = "cuda:0"


@pytest.mark.parametrize("E", [1, 15, 16, 17, 64, 65, 128, 129, 255, 256, 257])
@pytest.mark.parametrize("T", [1, 17, 130])
def test_route_rows_with_ties(E, T):
    print(f"route E={E} T={T}", flush=True)
    rng = np.random.default_rng(1000 * E + T)
    for k in sorted({1, min(E, 3), min(E, 16), min(E, 17)}):
        logits = np.round(rng.standard_normal((T, E)) * 2).astype(np.float32) / 2      # a handful of distinct scores
        logits[rng.random((T, E)) < 0.1] = -np.inf
        logits[:, rng.integers(0, E)] = 1.0                                              # a finite maximum in every row
        bias = np.round(rng.standard_normal(E)).astype(np.float32) if k != 3 else None
        idx, w = tq.tq_route(torch.from_numpy(logits).to(DEV), None if bias is None else torch.from_numpy(bias).to(DEV), k)
        torch.cuda.synchronize()
        ridx, rw = oracle.route(logits, bias, k)
        assert np.array_equal(idx.cpu().numpy(), ridx)
        assert np.max(np.abs(w.cpu().numpy() - rw)) <= 1e-6


@pytest.mark.parametrize("n", [257, 1023, 1024, 1025, 4095, 4096, 4097, 70001])
@pytest.mark.parametrize("E", [1, 130, 1024])
def test_permute_chunk_edges_with_invalid_index(n, E):
    print(f"permute n={n} E={E}", flush=True)
    rng = np.random.default_rng(n + E)
    idx = rng.integers(0, E, size=(n, 1)).astype(np.int32)
    bad = sorted({0, n // 2, n - 1})
    idx[bad[1]] = E
    idx[bad[2]] = -3
    err = torch.zeros(1, dtype=torch.int32, device=DEV)
    offsets, slot_of, src_of = tq.tq_permute(torch.from_numpy(idx).to(DEV), E, err_flag=err)
    torch.cuda.synchronize()
    assert int(err.item()) == 1
    flat = idx.reshape(-1)
    keep = (flat >= 0) & (flat < E)
    order = np.argsort(np.where(keep, flat, E), kind="stable")[:keep.sum()]
    slots = np.full(n, -1, np.int32)
    slots[order] = np.arange(len(order), dtype=np.int32)
    assert np.array_equal(offsets.cpu().numpy(), np.concatenate([[0], np.cumsum(np.bincount(flat[keep], minlength=E))]))
    assert np.array_equal(slot_of.cpu().numpy().reshape(-1), slots)
    assert np.array_equal(src_of.cpu().numpy().reshape(-1)[:len(order)], order)
