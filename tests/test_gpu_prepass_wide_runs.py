"""Pre-pass with four column tiles of t on either side of 96 row tiles (rows / 32 + experts), from where every XCD takes a run of
neighbouring tiles: with the contraction whole and cut into slices.  The bound is the medium batches'."""
import pytest

import paper_2605_09281_amd.binding as tq
from gpu_util import rel_err
from test_gpu_medium_batch import TOL_BF16, run, wide

pytestmark = pytest.mark.gpu

CASES = {
    "95": wide(3301, E=31, k=1, H=128, F=192, T=2079, r=64),
    "96": wide(3302, E=31, k=1, H=128, F=192, T=2080, r=64),
    "99_sliced_skewed": wide(3303, E=30, S=1, k=2, H=2048, F=320, T=726, r=48, zipf_s=1.1),
}


@pytest.mark.parametrize("name", list(CASES))
def test_prepass_of_four_column_tiles_by_runs(name):
    print(f"prepass wide runs {name}", flush=True)
    y, ref = run(CASES[name], tq.TQ_FLAG_FORCE_LARGE_TILE)
    assert rel_err(y.float().cpu().numpy(), ref) <= TOL_BF16
