"""The persistent tiled kernel's walk in strips of column blocks: strips of unequal width, under the deal by row tiles and under the deal by
column blocks, and the deal by column blocks where it leaves no fewer items.  Every item must be done exactly once: against the oracle
(bf16 activations and gate products, 2^-8 each, against the oracle's exact ones)."""
import pytest

import paper_2605_09281_amd.binding as tq
from gpu_util import rel_err
from test_gpu_medium_batch import TOL_BF16, run, wide

pytestmark = pytest.mark.gpu

CASES = {
    # gate/up: 13 column blocks, about nine row tiles an expert: strips of 7 and 6 by rows
    "rows_7_6": wide(3201, E=2, k=1, H=128, F=1664, T=1100),
    # gate/up: 97 column blocks, 13 or 12 in an XCD: strips of 7 and 6 or 6 and 6 by columns
    "cols_7_6": wide(3202, E=2, k=1, H=128, F=12416, T=1100),
    # gate/up: 32 column blocks, 15 or 16 row tiles: by columns with as many items as by rows
    "cols_level": wide(3203, E=2, k=1, H=256, F=4096, T=940),
    # down: 13 column blocks; gate/up: one, fewer than XCDs
    "down_7_6": wide(3204, E=2, k=1, H=3328, F=128, T=1100),
    "rows_7_6_dense_g128": wide(3205, E=2, k=1, H=256, F=1664, T=1100, g=128, bits=3, dense=True),
}


@pytest.mark.parametrize("name", list(CASES))
def test_strips_of_column_blocks(name):
    print(f"strips {name}", flush=True)
    y, ref = run(CASES[name], tq.TQ_FLAG_FORCE_LARGE_TILE)
    assert rel_err(y.float().cpu().numpy(), ref) <= TOL_BF16
