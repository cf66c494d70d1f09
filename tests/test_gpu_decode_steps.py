"""The decode kernels where their steps end: one to sixteen rows of a tile and one more, rows that take several rounds to stage, every group
size with contractions that leave waves idle or a last split short, ranks of one to all eight low-rank steps, dense codes in units of one and of two
chunks, and batches with the pre-pass by assignment and by tile.  Against the oracle, within four roundings to bf16 of the
output's scale (t, h and the output are rounded once each, 2^-9 relative, and chained through gate/up, SwiGLU and down)."""
import pytest
import torch

import paper_2605_09281_amd.binding as tq
from gpu_util import rel_err
from test_gpu_medium_batch import run, wide

pytestmark = pytest.mark.gpu

TOL = 4 * 2.0 ** -9
ONE = dict(E=1, k=1)
CASES = {f"{t}_rows_of_one_expert": wide(2800 + t, H=256, F=320, T=t, **ONE) for t in (1, 4, 5, 15, 16, 17)}
CASES.update({
    # 4096 wide: four rows a staging round
    "16_rows_of_4096": wide(2830, H=4096, F=128, g=128, T=16, **ONE),
    "9_rows_of_4096": wide(2831, H=4096, F=128, g=128, T=9, **ONE),
    "short_last_split": wide(2832, H=128, F=4224, T=5, r=24, **ONE),            # 4224 = 4096 + 128 indices
    "seven_of_eight_waves": wide(2833, H=256, F=3584, g=128, T=6, r=16, **ONE),
    "groups_of_32": wide(2834, H=192, F=2112, g=32, T=12, r=8),
    "groups_of_256": wide(2835, H=768, F=2304, g=256, T=12, r=40),
    "rank_64": wide(2836, H=320, F=448, T=12, r=64),
    "rank_0": wide(2837, H=320, F=448, T=12, r=0),
    "dense_3_units_of_one_chunk": wide(2838, H=320, F=2240, T=12, bits=3, dense=True),
    "dense_3_units_of_two": wide(2839, H=384, F=2304, g=128, T=12, bits=3, dense=True),
    "dense_2_units_of_one_chunk": wide(2840, H=320, F=448, T=12, bits=2, dense=True),
    "dense_2_units_of_two": wide(2841, H=2176, F=640, g=128, T=12, bits=2, dense=True),
    # workgroups of two and of four waves: 512 and 1024 indices are their last, with all eight low-rank steps among them
    "four_waves_groups_of_32": wide(2845, H=960, F=1024, g=32, T=12, r=64),
    "four_waves_dense_3": wide(2846, H=576, F=832, T=12, r=64, bits=3, dense=True),
    "two_waves_rank_64": wide(2847, H=512, F=512, g=128, T=16, r=64, **ONE),
    "four_waves_groups_of_256": wide(2848, H=1024, F=512, g=256, T=12, r=40),
    "many_experts_two_and_four_waves": wide(2849, E=40, k=4, H=512, F=1024, T=30, r=24),
    "256_rows_by_assignment": wide(2842, H=256, F=320, T=128, r=24),
    "258_rows_by_tile": wide(2843, H=256, F=320, T=129, r=24),
    "by_tile_40_experts": wide(2844, E=40, k=4, H=320, F=384, T=70, r=48, S=1),
})


@pytest.mark.parametrize("name", list(CASES))
def test_decode_kernels_at_the_ends_of_their_steps(name):
    print(f"decode steps {name}", flush=True)
    y, ref = run(CASES[name], tq.TQ_FLAG_FORCE_SKINNY)
    err = rel_err(y.float().cpu().numpy(), ref)
    print(f"   {err:.2e}")
    assert err <= TOL
    again, _ = run(CASES[name], tq.TQ_FLAG_FORCE_SKINNY)
    assert torch.equal(y.view(torch.int16), again.view(torch.int16))
