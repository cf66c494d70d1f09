"""tq_sketch_lowrank where every workgroup of a pass takes several steps: the loop that refills one register buffer while the
other is in work and reuses each half of the reduction buffer, on every shape of the pass, with even and odd numbers of
steps, a ragged last group of rows, and more ranks than pending deflations, so that passes that also store run through it."""
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


# columns, rows that all workgroups take in one step, pending deflations that fit; the shape of the pass (threads, float4
# columns per thread, rows at a time) follows from the columns alone
SHAPES = {
    "256x1x8": (64, 8192, 4), "256x1x8_full": (1024, 8192, 4), "256x2x4": (1028, 4096, 4), "256x4x2": (2052, 2048, 4),
    "512x4x2": (4100, 1024, 4), "1024x4x2": (8196, 512, 4), "1024x4x2_three_pending": (12672, 512, 3),
    "1024x4x2_two_pending": (16384, 512, 2), "1024x8x1": (16388, 256, 1), "1024x8x1_full": (32768, 256, 1),
}


@pytest.mark.parametrize("steps", [4, 5])
@pytest.mark.parametrize("name", list(SHAPES))
def test_several_steps_per_workgroup(name, steps):
    cols, per_step, pending = SHAPES[name]
    # some workgroups take `steps` whole steps, some one fewer, and one ends inside a group of rows (single-row groups: none)
    rows = (steps - 1) * per_step + per_step // 3 + (1 if per_step > 256 else 0)
    r, it = pending + 2, 1
    print(f"sketch {name} {rows}x{cols} r={r}", flush=True)
    gen = torch.Generator(device=DEV).manual_seed(rows + cols)
    n = lambda *shape: torch.randn(shape, generator=gen, device=DEV, dtype=torch.float64)
    # the same construction, and the same bound for the same reason, as in test_gpu_sketch.py
    W = ((n(rows, 24) * 0.7 ** torch.arange(24, device=DEV)) @ n(24, cols) + 0.05 * n(rows, cols)).float()
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
