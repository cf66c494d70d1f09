"""tq_sketch_lowrank on every shape of the pass over the matrix, with few and many steps a workgroup: up to as many steps as there are row
buffers nothing is requested twice (an instantiation of its own), beyond that a loop refills each buffer as soon as its rows are used, so what
matters is the number of steps modulo the number of buffers; some workgroups have a step less, and the last group of rows is ragged.  And matrices
so tall that a workgroup visits the vectors found so far more than once.  More than eight ranks, so that every count of earlier ranks that the
kernels are instantiated for occurs."""
import numpy as np
import pytest
import torch

from oracle.sketch_ref import sketch_lowrank
import paper_2605_09281_amd.binding as tq
from gpu_util import DEV

pytestmark = pytest.mark.gpu

# 2-norms: of a unit vector's difference, of Sigma's over the first, of the residual's over the matrix.  One rounding is
# 2^-24 = 6e-8 of a term; a product's entry carries a few of them (sums over threads, waves and workgroups in turn), and a rank
# sees those of the ranks before it divided by Sigma_i / Sigma_1 >= 0.05: 20 x 6e-8, and half as much again for the rest.
# (Measured: at most 3.1e-7.  One wrong row or column of W is 1e-3 and more of such a vector.)
TOL_NORM = 2e-6


def reference(W, it, S):
    """oracle.sketch_ref in fp64 on the device (matrices that would take numpy seconds each)."""
    W = W.double().clone()
    out = [], [], []
    for s in S.double():
        Q = W @ s
        for _ in range(it):
            Q = W @ (Q @ W)
            Q /= Q.norm()                 # the powers of a large matrix leave the fp32 range; U, Sigma, V do not depend on it
        P = Q @ W
        u, sigma, v = Q / Q.norm(), P.norm() / Q.norm(), P / P.norm()
        W.addr_(u, v, alpha=-float(sigma))
        for o, x in zip(out, (u, sigma, v)):
            o.append(x)
    return [torch.stack(o) for o in out] + [W]


def test_device_reference_is_the_oracle():
    rng = np.random.default_rng(5)
    W, S = rng.standard_normal((70, 36)), rng.standard_normal((3, 36))
    got = reference(torch.from_numpy(W).to(DEV), 2, torch.from_numpy(S).to(DEV))
    for a, b in zip(got, sketch_lowrank(W, 3, 2, S)):
        assert np.max(np.abs(a.cpu().numpy() - b)) <= 1e-10


# columns -> threads, rows in work at a time, row buffers, whether the column sums have 32 bits
def pass_shape(cols):
    nt = 256 if cols <= 4096 else 512 if cols <= 8192 else 1024
    rr = 8 if cols <= 1024 else 4 if cols <= 2048 else 1
    wide = cols > 16384
    return nt, rr, 2 if wide or rr > 1 else 3, wide


def steps_of(rows, cols):
    """Steps of the first workgroup, and whether another has one less."""
    nt, rr, _, wide = pass_shape(cols)
    wg = min(256 * 1024 // nt, max(256 if wide else 128, min(256, -(-rows // 16)), -(-rows // 32)), -(-rows // rr))
    groups = -(-rows // rr)
    return -(-groups // wg), groups % wg != 0


def rows_for(steps, cols):
    rr = pass_shape(cols)[1]
    for rows in range(100 + (rr > 1), 60000, 31):
        if steps_of(rows, cols) == (steps, steps > 1) and (rr == 1 or rows % rr):
            return rows
    raise AssertionError((steps, cols))


COLS = [64, 1024, 1028, 2052, 4100, 8196, 12672, 16384, 16388, 32768]


def check(rows, cols, r, it):
    print(f"sketch {rows}x{cols} r={r} it={it}", flush=True)
    gen = torch.Generator(device=DEV).manual_seed(rows + cols)
    n = lambda *shape: torch.randn(shape, generator=gen, device=DEV, dtype=torch.float64)
    k = min(24, cols)
    # the same construction, and the same bound for the same reason, as in test_gpu_sketch.py
    W = ((n(rows, k) * (0.7 if r < 9 else 0.85) ** torch.arange(k, device=DEV)) @ n(k, cols) + 0.05 * n(rows, cols)).float()
    S = n(r, cols).float()
    ref = reference(W, it, S)
    sigma1, norm = float(ref[1][0]), float(W.double().norm())
    U, sigma, V = tq.tq_sketch_lowrank(W, r, it, S)
    torch.cuda.synchronize()
    assert float(ref[1].min()) > 0.05 * sigma1            # every rank is a direction of the spectrum, not of noise
    err = [float((U - ref[0]).norm(dim=1).max()), float((sigma - ref[1]).abs().max()) / sigma1,
           float((V - ref[2]).norm(dim=1).max()), float((W - ref[3]).norm()) / norm]
    print("errors " + " ".join(f"{e:.1e}" for e in err), flush=True)
    assert max(err) <= TOL_NORM


@pytest.mark.parametrize("cols", COLS)
@pytest.mark.parametrize("more", [-1, 0, 1, 2, 3])
def test_steps_around_the_number_of_row_buffers(more, cols):
    nb = pass_shape(cols)[2]
    check(rows_for(nb + more, cols), cols, 6, 1)


@pytest.mark.parametrize("rows,cols", [(520, 1028), (300, 8196), (300, 16388), (5001, 68)])
@pytest.mark.parametrize("it", [0, 1])
def test_up_to_twelve_earlier_ranks(rows, cols, it):
    check(rows, cols, 13, it)
