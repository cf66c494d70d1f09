"""The lines between the decode kernels, the 32-row kernel and the large tilings, one case on each side: the batch without a
forced path is bit for bit the batch with that path forced, and agrees with the oracle (the bound of the medium batches:
bf16 activations and gate products, 2^-8 each, against the oracle's exact ones)."""
import pytest
import torch

import paper_2605_09281_amd.binding as tq
from gpu_util import DEV, rel_err
from test_gpu_medium_batch import TOL_BF16, run, wide

pytestmark = pytest.mark.gpu

DECODE, SMALL, LARGE = tq.TQ_FLAG_FORCE_SKINNY, tq.TQ_FLAG_FORCE_SMALL_TILE, tq.TQ_FLAG_FORCE_LARGE_TILE
CASES = {
    # the rows decide, neither the number of assignments nor the shape of the layer
    "324_assignments": (wide(2702, E=41, k=4, H=256, F=384, T=81), DECODE),
    "width_past_6_times_height": (wide(2704, E=8, H=256, F=1600, T=20), DECODE),
    "wide_18_assignments": (wide(2706, E=8, H=256, F=1600, T=9), DECODE),
    "wide_dense_codes": (wide(2707, E=8, H=256, F=1600, T=9, bits=3, dense=True), DECODE),
    "10_rows_of_16_experts": (wide(2710, E=16, H=256, F=384, T=87), DECODE),
    "11_rows_of_16_experts": (wide(2711, E=16, H=256, F=384, T=88), SMALL),
    "8_rows_of_41_experts": (wide(2712, E=41, k=4, H=256, F=384, T=82), DECODE),
    "past_8_rows_of_41_experts": (wide(2713, E=41, k=4, H=256, F=384, T=83), SMALL),
    "1524_by_1024_by_1280": (wide(2708, H=1024, F=1280, T=762), SMALL),
    "1526_by_1024_by_1280": (wide(2709, H=1024, F=1280, T=763), LARGE),
    # at most 4096 assignments, a short F: by the values of a plane, assignments x H
    "planes_of_800000": (wide(2714, E=8, H=640, F=640, T=625), SMALL),
    "planes_past_800000": (wide(2715, E=8, H=640, F=640, T=626), LARGE),
    "planes_past_800000_F_1216": (wide(2716, E=8, H=640, F=1216, T=640), LARGE),
    "planes_past_800000_F_1280": (wide(2717, E=8, H=640, F=1280, T=640), SMALL),
    "4096_assignments": (wide(2718, E=8, H=256, F=320, T=2048), LARGE),
    "4098_assignments": (wide(2719, E=8, H=256, F=320, T=2049), SMALL),
}


@pytest.mark.parametrize("name", list(CASES))
def test_each_side_of_the_lines_between_the_paths(name):
    print(f"path lines {name}", flush=True)
    cfg, flag = CASES[name]
    y, ref = run(cfg, 0)
    assert rel_err(y.float().cpu().numpy(), ref) <= TOL_BF16
    forced, _ = run(cfg, flag)
    assert torch.equal(y.view(torch.int16), forced.view(torch.int16))


@pytest.mark.parametrize("T", [81, 101, 120])
def test_benchmark_layer_stays_on_the_decode_kernels(T):
    """60 experts of 2048 x 1408, groups of 64, rank 64, up to 8 rows an expert: the decode kernels' output to the bit."""
    E, k, H, F, g, r = 60, 4, 2048, 1408, 64, 64
    print(f"benchmark layer T {T}", flush=True)
    gen = torch.Generator(device=DEV).manual_seed(T)

    def half(*shape, scale):
        return (torch.randn(shape, generator=gen, device=DEV) * scale).half().view(torch.int16)

    codes = torch.randint(0, 16, (E, 3, H * F), generator=gen, device=DEV, dtype=torch.uint8)
    scale, zero = half(E, 3, H * F // g, scale=0.005), torch.full((E, 3, H * F // g), 7.5, device=DEV).half().view(torch.int16)
    A, B = half(E, (2 * H + F) * r, scale=0.01), half(E, (2 * F + H) * r, scale=0.01)
    x = torch.randn((T, H), generator=gen, device=DEV).bfloat16()
    idx, w = tq.tq_route(torch.randn((T, E), generator=gen, device=DEV), None, k)
    packed = tq.tq_pack_weights(tq.make_desc(E, 0, k, H, F, g, 4, r, tq.TQ_ACT_BF16), codes, scale, zero, A, B)
    ys = [tq.tq_moe_forward(tq.make_desc(E, 0, k, H, F, g, 4, r, tq.TQ_ACT_BF16, flags), packed, x, idx, w) for flags in (0, DECODE)]
    assert bool(torch.isfinite(ys[0].float()).all()) and float(ys[0].float().abs().max()) > 0
    assert torch.equal(ys[0].view(torch.int16), ys[1].view(torch.int16))
