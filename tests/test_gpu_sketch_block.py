"""tq_sketch_lowrank where the first products of up to 16 ranks come from one pair of block products, and where the deflations are applied
to the vectors: batches of 16 ranks and what remains, few rows (contraction cut in parts), many rows (slabs), no power iterations on
either side of the size that takes the block, spectra whose subtractions cancel many digits, extreme scales, more ranks than the matrix has."""
import pytest
import torch

import paper_2605_09281_amd.binding as tq
from gpu_util import DEV
from test_gpu_sketch_steps import TOL_NORM, reference

pytestmark = pytest.mark.gpu


def matrix(rows, cols, decay, noise, seed):
    gen = torch.Generator(device=DEV).manual_seed(seed)
    n = lambda *shape: torch.randn(shape, generator=gen, device=DEV, dtype=torch.float64)
    k = min(rows, cols, 40)
    return ((n(rows, k) * decay ** torch.arange(k, device=DEV)) @ n(k, cols) + noise * n(rows, cols)), n


def errors(W, S, it):
    """2-norm errors of U, Sigma (relative to itself), V and the residual (relative to the matrix)."""
    ref = reference(W, it, S)
    norm = float(W.double().norm())
    U, sigma, V = tq.tq_sketch_lowrank(W, S.shape[0], it, S)
    torch.cuda.synchronize()
    return [float((U - ref[0]).norm(dim=1).max()), float(((sigma - ref[1]) / ref[1]).abs().max()),
            float((V - ref[2]).norm(dim=1).max()), float((W - ref[3]).norm()) / norm]


@pytest.mark.parametrize("rows,cols,r,it", [(40, 1028, 17, 1), (33, 16384, 16, 2), (31, 12, 3, 1), (5000, 2052, 18, 0), (700, 2052, 4, 0),
                                            (2100, 4100, 33, 1), (65, 68, 16, 3), (20000, 64, 16, 1), (16, 16384, 5, 0)])
def test_blocks_of_ranks(rows, cols, r, it):
    print(f"sketch {rows}x{cols} r={r} it={it}", flush=True)
    W, n = matrix(rows, cols, 0.9, 0.05, rows + cols + r)
    e = errors(W.float(), n(r, cols).float(), it)
    print("errors " + " ".join(f"{x:.1e}" for x in e), flush=True)
    # the bound of test_gpu_sketch_steps.py (32-bit sums; here they have 64 bits and the rounding of the results remains)
    assert max(e) <= TOL_NORM


@pytest.mark.parametrize("it", [0, 1, 2])
@pytest.mark.parametrize("scale", [1.0, 1e-15, 1e12])
def test_cancellation_over_five_digits(it, scale):
    """Singular values fall by 2 per rank: the 16th is 3e-5 of the first, so W^T W s cancels nine digits.  32-bit vectors would be off by
    6e-8 x 3e4 = 2e-3; in 64 bits what is left is the rounding of the results (bound as above)."""
    W, n = matrix(1500, 1200, 0.5, 1e-7, 5)
    e = errors((W * scale).float(), n(16, 1200).float(), it)
    print("errors " + " ".join(f"{x:.1e}" for x in e), flush=True)
    assert max(e) <= TOL_NORM


@pytest.mark.parametrize("it", [0, 2])
@pytest.mark.parametrize("scale", [1e-15, 1e12])
def test_scales_where_the_column_sums_have_32_bits(it, scale):
    """Past 16384 columns: the first q of a rank has the length of W s, and the column sums that of W^T W s."""
    W, n = matrix(300, 17000, 0.7, 0.05, 6)
    e = errors((W * scale).float(), n(6, 17000).float(), it)
    print("errors " + " ".join(f"{x:.1e}" for x in e), flush=True)
    assert max(e) <= TOL_NORM


@pytest.mark.parametrize("rows,cols", [(3, 64), (64, 4), (2, 17000)])
@pytest.mark.parametrize("it", [0, 2])
def test_more_ranks_than_the_matrix_has(rows, cols, it):
    """The ranks past the last one are zero vectors or directions of what rounding left: nothing of the matrix may come back."""
    W, n = matrix(rows, cols, 0.9, 0.0, rows + cols)
    W = W.float()
    full, r = min(rows, cols), min(rows, cols) + 3
    W0 = W.double()
    U, sigma, V = tq.tq_sketch_lowrank(W, r, it, n(r, cols).float())
    torch.cuda.synchronize()
    assert all(bool(torch.isfinite(t).all()) for t in (U, sigma, V, W))
    assert float(sigma[full:].max()) <= 1e-5 * float(sigma[0])
    rec = (U.double().T * sigma.double()) @ V.double() + W.double()
    assert float((rec - W0).norm()) <= TOL_NORM * float(W0.norm())
    assert float(W.double().norm()) <= 1e-5 * float(W0.norm())
