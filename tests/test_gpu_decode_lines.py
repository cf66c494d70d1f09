"""The lines up to which layers of fewer than 16 experts stay on the decode kernels, by the size of their weights, one case on each side: the
batch without a forced path is bit for bit the batch with that path forced, and agrees with the oracle (bf16 activations and gate
products, 2^-8 each, against the oracle's exact ones)."""
import pytest
import torch

import paper_2605_09281_amd.binding as tq
from gpu_util import rel_err
from test_gpu_medium_batch import TOL_BF16, run, wide

pytestmark = pytest.mark.gpu

DECODE, SMALL = tq.TQ_FLAG_FORCE_SKINNY, tq.TQ_FLAG_FORCE_SMALL_TILE
CASES = {
    # (E + S) H F up to 10 M: 32 rows an expert
    "32_rows_of_15": (wide(3101, E=15, H=256, F=384, T=240), DECODE),
    "past_32_rows_of_15": (wide(3102, E=15, H=256, F=384, T=241), SMALL),
    "32_rows_with_a_shared_expert": (wide(3103, E=6, S=1, H=256, F=384, T=74), DECODE),
    "32_rows_dense_codes": (wide(3104, E=8, H=256, F=384, T=128, bits=3, dense=True), DECODE),
    "past_32_rows_dense_codes": (wide(3105, E=8, H=256, F=384, T=129, bits=3, dense=True), SMALL),
    # 10.5 M: 20 rows
    "20_rows_past_10M": (wide(3106, E=8, H=512, F=2560, T=80), DECODE),
    "past_20_rows_past_10M": (wide(3107, E=8, H=512, F=2560, T=81), SMALL),
    # 31 M: 16 rows
    "16_rows_past_30M": (wide(3108, E=4, H=1024, F=7616, g=64, T=32), DECODE),
    "past_16_rows_past_30M": (wide(3109, E=4, H=1024, F=7616, g=64, T=33), SMALL),
    "16_experts_keep_their_line": (wide(3110, E=16, H=256, F=384, T=90), SMALL),
}


@pytest.mark.parametrize("name", list(CASES))
def test_each_side_of_the_decode_lines_of_small_layers(name):
    print(f"decode lines {name}", flush=True)
    cfg, flag = CASES[name]
    y, ref = run(cfg, 0)
    assert rel_err(y.float().cpu().numpy(), ref) <= TOL_BF16
    forced, _ = run(cfg, flag)
    assert torch.equal(y.view(torch.int16), forced.view(torch.int16))
