"""The lines between the decode kernels, the 32-row kernel and the large tilings, one case on each side: the batch without a
forced path is bit for bit the batch with that path forced, and agrees with the oracle (the bound of the medium batches:
bf16 activations and gate products, 2^-8 each, against the oracle's exact ones)."""
import pytest
import torch

import paper_2605_09281_amd.binding as tq
from gpu_util import rel_err
from test_gpu_medium_batch import TOL_BF16, run, wide

pytestmark = pytest.mark.gpu

DECODE, SMALL, LARGE = tq.TQ_FLAG_FORCE_SKINNY, tq.TQ_FLAG_FORCE_SMALL_TILE, tq.TQ_FLAG_FORCE_LARGE_TILE
CASES = {
    "320_assignments": (wide(2701, E=41, k=4, H=256, F=384, T=80), DECODE),
    "324_assignments": (wide(2702, E=41, k=4, H=256, F=384, T=81), SMALL),
    "width_6_times_height": (wide(2703, E=8, H=256, F=1536, T=20), DECODE),
    "width_past_6_times_height": (wide(2704, E=8, H=256, F=1600, T=20), SMALL),
    "wide_16_assignments": (wide(2705, E=8, H=256, F=1600, T=8), DECODE),
    "wide_18_assignments": (wide(2706, E=8, H=256, F=1600, T=9), SMALL),
    "wide_dense_codes": (wide(2707, E=8, H=256, F=1600, T=9, bits=3, dense=True), DECODE),
    "1906_by_1024_by_1024": (wide(2708, H=1024, F=1024, T=953), SMALL),
    "1908_by_1024_by_1024": (wide(2709, H=1024, F=1024, T=954), LARGE),
}


@pytest.mark.parametrize("name", list(CASES))
def test_each_side_of_the_lines_between_the_paths(name):
    print(f"path lines {name}", flush=True)
    cfg, flag = CASES[name]
    y, ref = run(cfg, 0)
    assert rel_err(y.float().cpu().numpy(), ref) <= TOL_BF16
    forced, _ = run(cfg, flag)
    assert torch.equal(y.view(torch.int16), forced.view(torch.int16))
