"""Pre-pass of the tiled kernels on either side of 768 row tiles (rows / 32 + experts), from where every XCD takes a run of neighbouring
tiles: tile counts that are and are not a multiple of eight, group counts that do not fill a chunk of four, the widths of t whose
factor fragments come in two halves.  The bound is the medium batches'."""
import pytest

import paper_2605_09281_amd.binding as tq
from gpu_util import rel_err
from test_gpu_medium_batch import TOL_BF16, run, wide

pytestmark = pytest.mark.gpu

SMALL, LARGE = tq.TQ_FLAG_FORCE_SMALL_TILE, tq.TQ_FLAG_FORCE_LARGE_TILE
CASES = {
    "767": (wide(2901, E=5, k=1, H=128, F=192, T=24400, g=64, r=8), SMALL),
    "768": (wide(2902, E=5, k=1, H=128, F=192, T=24416, g=64, r=8), SMALL),
    "768_skewed_one_group": (wide(2903, E=8, k=1, H=128, F=256, T=24320, g=128, r=32, zipf_s=1.2), LARGE),
    "800_four_column_tiles": (wide(2904, E=32, S=1, k=2, H=192, F=320, T=8184, g=64, r=64), LARGE),
}


@pytest.mark.parametrize("name", list(CASES))
def test_prepass_by_runs_of_tiles(name):
    print(f"prepass runs {name}", flush=True)
    cfg, flags = CASES[name]
    y, ref = run(cfg, flags)
    assert rel_err(y.float().cpu().numpy(), ref) <= TOL_BF16
