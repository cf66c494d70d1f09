"""What the tiled kernels read beside the blob (fp16 fragments of fp8 factors, zero-point fragments of dense codes) is derived by
workgroups in the permutation's launch: in the single-wave one, with and without the routing, and in the placing one after its own
count and after the histogram; ranges of workgroups that end inside a workgroup of eight waves.  Against the oracle, in a workspace that held other
bytes before; the bound is the one of the fp8 tests (activations and gate products rounded to bf16, four roundings of 2^-9)."""
import pytest
import torch

import oracle
from synth import make_layer_fp8, make_logits, make_x
import paper_2605_09281_amd.binding as tq
from gpu_util import DEV, rel_err, x_device
from test_gpu_fp8_factors import REG_BF16, desc_fp8, fcfg, pack_gpu

pytestmark = pytest.mark.gpu

CASES = {
    "single_wave": (fcfg(2801, E=5, S=1, bits=3, dense=True, r=24, T=40), False),
    "single_wave_routed": (fcfg(2802, E=5, S=1, bits=3, dense=True, r=24, T=40), True),
    "placing_counts_itself": (fcfg(2803, E=7, bits=2, dense=True, r=16, T=333), False),
    "placing_after_histogram": (fcfg(2804, E=9, k=3, H=64, F=64, bits=3, dense=True, r=8, T=1600), True),
}


@pytest.mark.parametrize("name", list(CASES))
def test_parts_beside_the_blob(name):
    print(f"prep {name}", flush=True)
    cfg, routed = CASES[name]
    fl, x = make_layer_fp8(cfg), make_x(cfg)
    logits, bias = make_logits(cfg)
    packed = pack_gpu(fl)
    lg, bs = torch.from_numpy(logits).to(DEV), None if bias is None else torch.from_numpy(bias).to(DEV)
    idx, w = tq.tq_route(lg, bs, cfg.k)
    desc = desc_fp8(cfg, flags=tq.TQ_FLAG_FORCE_SMALL_TILE)
    ws = torch.empty(tq.tq_moe_workspace_size(desc, cfg.T), dtype=torch.uint8, device=DEV)
    ref = oracle.moe_forward_fp8(cfg, fl.codes, fl.scale, fl.zero, fl.a8_list(), fl.b8_list(), fl.sigma, x, idx.cpu().numpy(),
                                 w.cpu().numpy())
    for fill in (0x5A, 0xFF):
        ws.fill_(fill)
        xd = x_device(x, tq.TQ_ACT_BF16)
        if routed:
            y = torch.empty_like(xd)
            tq.tq_route_moe_forward(desc, packed, xd, lg, bs, torch.empty_like(idx), torch.empty_like(w), y, ws)
        else:
            y = tq.tq_moe_forward(desc, packed, xd, idx, w, workspace=ws)
        torch.cuda.synchronize()
        assert int(ws[:4].view(torch.int32).item()) == 0
        assert rel_err(y.float().cpu().numpy(), ref) <= REG_BF16
