"""tq_permute and a layer past the number of counts (chunks of 1024 assignments x experts) at which the counts are added up by a
launch of their own: on both sides of that line, with expert numbers that do and do not fill the scan's workgroups, one
expert, a ragged last run of chunks and invalid indices, bit for bit against a stable sort; and the time of a large batch
against that of a quarter of it."""
import pytest
import torch

import paper_2605_09281_amd.binding as tq
from gpu_util import DEV, rel_err
from test_gpu_medium_batch import TOL_BF16, run, wide

pytestmark = pytest.mark.gpu

LINE = 32768      # counts


def check_permute(n, E, seed):
    gen = torch.Generator(device=DEV).manual_seed(seed)
    idx = torch.randint(0, E, (n, 1), generator=gen, device=DEV, dtype=torch.int32)
    idx[n // 2], idx[n - 1] = E, -3
    err = torch.zeros(1, dtype=torch.int32, device=DEV)
    n_ws = tq.lib().tq_permute_workspace_size(n, E, 1)
    ws = torch.full((n_ws + 4096,), 0x5A, dtype=torch.uint8, device=DEV)      # guard bytes behind the workspace
    offsets, slot_of, src_of = (torch.empty(m, dtype=torch.int32, device=DEV) for m in (E + 1, n, n))
    rc = tq.lib().tq_permute(idx.data_ptr(), n, E, 1, offsets.data_ptr(), slot_of.data_ptr(), src_of.data_ptr(), err.data_ptr(),
                             ws.data_ptr(), n_ws, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert rc == 0 and int(err.item()) == 1
    assert int((ws[n_ws:] != 0x5A).sum()) == 0
    flat = idx.view(-1).long()
    key = torch.where((flat >= 0) & (flat < E), flat, E)
    order = torch.sort(key, stable=True).indices
    counts = torch.bincount(key, minlength=E + 1)
    kept = n - int(counts[E])
    assert kept == n - 2
    slots = torch.full((n,), -1, dtype=torch.int32, device=DEV)
    slots[order[:kept]] = torch.arange(kept, dtype=torch.int32, device=DEV)
    assert torch.equal(offsets.long()[1:], torch.cumsum(counts[:E], 0)) and int(offsets[0]) == 0
    assert torch.equal(slot_of, slots)
    assert torch.equal(src_of[:kept].long(), order[:kept])


@pytest.mark.parametrize("E", [1, 5, 8, 33, 130, 1000, 1024])
@pytest.mark.parametrize("side", ["below", "at", "past"])
def test_permute_around_the_scan_line(E, side):
    at = -(-LINE // E)                                    # the first number of chunks with a scan
    chunks = {"below": at - 1, "at": at, "past": at + 9}[side]
    print(f"permute E={E} chunks={chunks}", flush=True)
    check_permute(1024 * chunks - (0 if side == "at" else 1001), E, 1000 * E + chunks)


def test_permute_with_few_chunks_per_run_and_with_many():
    check_permute(40 * 1024 + 17, 1024, 1)               # 41 chunks over 32 runs: two each, the last runs empty
    check_permute(1500 * 1024 + 17, 1024, 2)             # 47 chunks per run: whole batches of eight and a remainder


def test_layer_whose_permutation_scans():
    cfg = wide(2501, E=1000, S=2, k=8, H=64, F=64, T=4230, g=64, r=8)      # 34 chunks of 1000 experts
    y, ref = run(cfg, 0)
    assert rel_err(y.float().cpu().numpy(), ref) <= TOL_BF16


def us(f, n=3):
    f()
    torch.cuda.synchronize()
    times = []
    for _ in range(n):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        f()
        b.record()
        b.synchronize()
        times.append(1000 * a.elapsed_time(b))
    return min(times)


def test_permutation_time_grows_linearly():
    """Four times the assignments take about four times as long (119 / 38 us measured).  With every workgroup adding up all
    counts it is sixteen times (4495 / 314 us measured); the bound lies at the middle of the two, as ratios."""
    E, t = 1024, {}
    for n in (1 << 20, 1 << 22):
        idx = torch.randint(0, E, (n, 1), device=DEV, dtype=torch.int32)
        t[n] = us(lambda: tq.tq_permute(idx, E))
    print(f"permute 1 M / 4 M assignments of {E} experts: {t[1 << 20]:.0f} / {t[1 << 22]:.0f} us", flush=True)
    assert t[1 << 22] <= 8 * t[1 << 20]
