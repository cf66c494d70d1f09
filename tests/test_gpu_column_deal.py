"""One-workgroup-per-item tiled kernels on a number of row tiles that does not divide over the eight XCDs: the column blocks
are then dealt to the XCDs.  Column counts that are a multiple of eight and that are not, 32-row tiles and 64-row tiles with
the contraction split into planes."""
import pytest

import paper_2605_09281_amd.binding as tq
from gpu_util import rel_err
from test_gpu_medium_batch import TOL_BF16, run, wide

pytestmark = pytest.mark.gpu

CASES = {
    "11_blocks_9_tiles": (wide(2431, E=9, k=1, H=2816, F=1408, T=60), tq.TQ_FLAG_FORCE_SMALL_TILE),
    "8_blocks_9_tiles_g128": (wide(2432, E=9, k=2, H=2048, F=1024, T=100, g=128), tq.TQ_FLAG_FORCE_SMALL_TILE),
    "8_blocks_split": (wide(2433, E=9, k=2, H=2048, F=4096, T=100, g=128), tq.TQ_FLAG_FORCE_LARGE_TILE),
    "8_blocks_split_ragged_tiles": (wide(2434, E=6, k=1, H=2048, F=4096, T=420), tq.TQ_FLAG_FORCE_LARGE_TILE),
}


@pytest.mark.parametrize("name", list(CASES))
def test_column_blocks_dealt_to_the_xcds(name):
    print(f"column deal {name}", flush=True)
    cfg, flags = CASES[name]
    y, ref = run(cfg, flags)
    assert rel_err(y.float().cpu().numpy(), ref) <= TOL_BF16
