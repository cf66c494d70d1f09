"""tq_pack_weights / tq_unpack_weights where the pack kernels' spans end unevenly: eight 64-wide chunks and 64 groups per
workgroup, with one chunk or group more, one less and a short last span.  Byte for byte against oracle/pack_ref.py."""
import numpy as np
import pytest
import torch

from oracle import pack_ref
from synth import LayerConfig, make_layer
import paper_2605_09281_amd.binding as tq
from gpu_util import DEV, desc_of, pack_layer_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,F,g,bits,dense", [(64, 576, 32, 4, False), (448, 512, 64, 4, False), (2112, 64, 32, 4, False),
                                              (2048, 1088, 64, 3, False), (576, 704, 64, 3, True), (1088, 448, 64, 2, True)])
def test_pack_spans(H, F, g, bits, dense):
    cfg = LayerConfig(890, "spans", E=2, S=0, k=1, H=H, F=F, T=1, g=g, r=0, bits=bits, dense=dense)
    layer = make_layer(cfg, workers=2)
    packed = pack_layer_gpu(layer)
    assert np.array_equal(packed.cpu().numpy()[256:], pack_ref.pack_layer(layer))
    codes = torch.full(layer.codes.shape, 255, dtype=torch.uint8, device=DEV)
    scale = torch.zeros(layer.scale.shape, dtype=torch.int16, device=DEV)
    zero = torch.zeros_like(scale)
    tq.tq_unpack_weights(desc_of(cfg), packed, codes, scale, zero)
    torch.cuda.synchronize()
    assert np.array_equal(codes.cpu().numpy(), layer.codes)
    assert np.array_equal(scale.cpu().numpy().view(np.uint16), layer.scale)
    assert np.array_equal(zero.cpu().numpy().view(np.uint16), layer.zero)
