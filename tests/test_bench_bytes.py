"""The byte count behind the decomposition's bandwidth in bench.py, against counts made by hand from the kernels."""
import pytest

from bench import sketch_streams


@pytest.mark.parametrize("rows,cols,r,it,reads,writes", [
    (16384, 12672, 16, 2, 2 + 32 + 1, 1),               # one batch with block products
    (16384, 12672, 32, 2, 2 * (2 + 32 + 1), 2),         # the residual is stored after every 16 ranks
    (16384, 12672, 18, 2, (2 + 32 + 1) + (6 + 1), 2),   # two ranks left: three passes each
    (16384, 12672, 16, 0, 2 + 1, 1),                    # no iterations: the block products are all
    (1024, 1024, 8, 0, 8 + 1, 1),                       # ... too small for them: a pass per rank
    (1000000, 4, 6, 1, (2 + 4 + 1) + (4 + 1), 2),       # no batch has more ranks than the matrix
    (4096, 20000, 16, 2, 48 + 1, 1),                    # 32-bit column sums: it + 1 passes per rank
    (100, 40000, 3, 2, 3 * 6 + 1, 3),                   # one stream per product, the deflation stored per rank
])
def test_sketch_streams(rows, cols, r, it, reads, writes):
    assert sketch_streams(rows, cols, r, it) == (reads, writes)
