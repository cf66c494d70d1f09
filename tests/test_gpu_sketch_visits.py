"""tq_sketch_lowrank on matrices so tall that a workgroup of a pass takes more rows than it keeps vectors' entries for (1024 on workgroups of
256 threads, 256 on wider ones): it then visits the u_ij found so far again, refills its row buffers and adds to the sums it carries."""
import pytest
import torch

from test_gpu_sketch_steps import check

pytestmark = pytest.mark.gpu


# rows that all workgroups of a width keep entries for, and a ragged few more for some of them
@pytest.mark.parametrize("rows,cols", [(1048576 + 4099, 4), (1048576 + 4099, 1028), (2 * 1048576 + 70, 68), (1048576 + 300, 2052), (131072 + 700, 4100),
                                       (65536 + 300, 8196), (2 * 65536 + 100, 8196), (65536 + 300, 16388)])
def test_more_rows_than_one_visit_takes(rows, cols):
    check(rows, cols, min(cols - 1, 5), 1)      # five ranks: passes with none, and with up to four, found before
    torch.cuda.empty_cache()
