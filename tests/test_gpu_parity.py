"""GPU parity tests: the HIP library, called through its C ABI, against the CPU oracle on the same
seeded inputs.  Integer work (routing indices, permutation, pack/unpack) is bit-exact; floating
point within max|gpu-oracle|/max|oracle| <= 2e-2 (bf16 activations) and <= 1e-5 (fp32 debug path)."""
import numpy as np
import pytest
import torch

import oracle
from oracle import pack_ref
from synth import CONFIGS, LayerConfig, make_layer, make_x, make_logits
import paper_2605_09281_amd.binding as tq
from gpu_util import DEV, dev16, desc_of, pack_layer_gpu, x_device, rel_err

pytestmark = pytest.mark.gpu

TOL_BF16 = 2e-2
TOL_FP32 = 1e-5


def small_cfg(cfg_id, **kw):
    base = dict(name="s", E=4, S=0, k=2, H=128, F=192, T=37, g=64, r=8, bits=4)
    base.update(kw)
    return LayerConfig(cfg_id, **base)


SMALL = {
    "base": small_cfg(201),
    "shared": small_cfg(202, S=2, E=6, k=3, T=50),
    "rank0": small_cfg(203, r=0),
    "int3_g32": small_cfg(204, bits=3, g=32, r=20, H=192, F=128, T=21),
    "ragged": small_cfg(205, E=16, k=4, H=256, F=320, T=150, g=64, r=32),   # rows/expert ~37: several 32-row tiles
    "one_token": small_cfg(206, T=1, E=8, k=2),
    "g128_r64": small_cfg(207, H=256, F=384, g=128, r=64, E=5, k=5, T=40),
    "g64_r64": small_cfg(208, H=256, F=192, g=64, r=64, E=6, k=3, T=90),       # four column tiles of t in the gate/up pre-pass
    "g32_r40": small_cfg(209, H=192, F=256, g=32, r=40, E=4, k=2, T=70),       # three (r16 = 48), groups of 32
}

_cache = {}


def get_layer(cfg):
    if cfg.cfg_id not in _cache:
        _cache[cfg.cfg_id] = make_layer(cfg, workers=8)
    return _cache[cfg.cfg_id]


# ------------------------------------------------------------------ pack / unpack
@pytest.mark.parametrize("name", ["base", "shared", "rank0", "int3_g32", "g128_r64"])
def test_pack_is_byte_exact_and_unpack_inverts(name):
    cfg = SMALL[name]
    layer = get_layer(cfg)
    packed = pack_layer_gpu(layer)
    body = packed.cpu().numpy()[256:]
    ref = pack_ref.pack_layer(layer)
    assert body.size == ref.size
    assert np.array_equal(body, ref)
    # inverse
    desc = desc_of(cfg)
    codes = torch.full(layer.codes.shape, 255, dtype=torch.uint8, device=DEV)
    scale = torch.zeros(layer.scale.shape, dtype=torch.int16, device=DEV)
    zero = torch.zeros_like(scale)
    A = torch.zeros(layer.A.shape, dtype=torch.int16, device=DEV) if cfg.r else None
    B = torch.zeros(layer.B.shape, dtype=torch.int16, device=DEV) if cfg.r else None
    tq.tq_unpack_weights(desc, packed, codes, scale, zero, A, B)
    torch.cuda.synchronize()
    assert np.array_equal(codes.cpu().numpy(), layer.codes)
    assert np.array_equal(scale.cpu().numpy().view(np.uint16), layer.scale)
    assert np.array_equal(zero.cpu().numpy().view(np.uint16), layer.zero)
    if cfg.r:
        assert np.array_equal(A.cpu().numpy().view(np.uint16), layer.A)
        assert np.array_equal(B.cpu().numpy().view(np.uint16), layer.B)


def test_pack_every_nibble_position_and_range_flag():
    cfg = small_cfg(210, E=1, k=1, H=64, F=64, g=64, r=0)
    layer = get_layer(cfg)
    import copy
    l2 = copy.copy(layer)
    codes = np.zeros_like(layer.codes)
    flat = codes.reshape(-1)
    flat[:] = (np.arange(flat.size) * 7 + (np.arange(flat.size) // 64)) % 16     # every position sees every code
    l2.codes = codes
    packed = pack_layer_gpu(l2)
    assert np.array_equal(packed.cpu().numpy()[256:], pack_ref.pack_layer(l2))
    # a code above qmax raises the device flag (bits = 3 -> qmax 7)
    desc = tq.make_desc(1, 0, 1, 64, 64, 64, 3, 0)
    err = torch.zeros(1, dtype=torch.int32, device=DEV)
    tq.tq_pack_weights(desc, torch.from_numpy(codes).to(DEV), dev16(layer.scale), dev16(layer.zero), err_flag=err)
    torch.cuda.synchronize()
    assert int(err.item()) & 1
    err.zero_()
    tq.tq_pack_weights(desc, torch.from_numpy(codes % 8).to(DEV), dev16(layer.scale), dev16(layer.zero), err_flag=err)
    torch.cuda.synchronize()
    assert int(err.item()) == 0


# ------------------------------------------------------------------ routing
@pytest.mark.parametrize("T,E,k,use_bias,seed", [(64, 8, 2, False, 0), (16, 8, 2, True, 1), (333, 64, 6, True, 2),
                                                  (1024, 60, 4, False, 3), (2000, 128, 8, True, 4), (5, 5, 5, False, 5),
                                                  (9, 130, 1, False, 6), (3, 1000, 64, True, 7), (1, 2, 1, False, 8)])
def test_route_indices_bit_exact_weights_close(T, E, k, use_bias, seed):
    rng = np.random.default_rng(seed)
    logits = rng.standard_normal((T, E)).astype(np.float32)
    bias = (-1.1 * np.log(rng.permutation(E) + 1.0)).astype(np.float32) if use_bias else None
    idx, w = tq.tq_route(torch.from_numpy(logits).to(DEV), None if bias is None else torch.from_numpy(bias).to(DEV), k)
    torch.cuda.synchronize()
    ridx, rw = oracle.route(logits, bias, k)
    assert np.array_equal(idx.cpu().numpy(), ridx)
    got = w.cpu().numpy()
    assert np.max(np.abs(got - rw)) <= 1e-6
    assert np.max(np.abs(got.astype(np.float64).sum(axis=1) - 1.0)) <= 1e-6


def test_route_ties_and_degenerate_rows():
    logits = np.array([[1, 3, 3, 0, 3, 1, -2, 3],
                       [0.5] * 8,
                       [-np.inf, 0, -np.inf, 0, 1, 1, 1, -np.inf],
                       [7, 6, 5, 4, 3, 2, 1, 0]], dtype=np.float32)
    for k in (1, 3, 4, 8):
        idx, w = tq.tq_route(torch.from_numpy(logits).to(DEV), None, k)
        torch.cuda.synchronize()
        ridx, rw = oracle.route(logits, None, k)
        if k == 8:      # rows with -inf scores: exp(-inf) = 0 weights, order of the -inf entries by index
            assert np.array_equal(idx.cpu().numpy(), ridx)
        else:
            assert np.array_equal(idx.cpu().numpy(), ridx)
        assert np.max(np.abs(w.cpu().numpy() - rw)) <= 1e-6
    # the configs' own routers
    for c in (1, 3, 5):
        cfg = CONFIGS[c]
        lg, b = make_logits(cfg)
        idx, w = tq.tq_route(torch.from_numpy(lg).to(DEV), None if b is None else torch.from_numpy(b).to(DEV), cfg.k)
        torch.cuda.synchronize()
        ridx, rw = oracle.route(lg, b, cfg.k)
        assert np.array_equal(idx.cpu().numpy(), ridx)
        assert np.max(np.abs(w.cpu().numpy() - rw)) <= 1e-6


# ------------------------------------------------------------------ permutation
@pytest.mark.parametrize("T,E,k,seed", [(1, 4, 2, 0), (16, 8, 2, 1), (257, 60, 4, 2), (8192, 128, 8, 3), (3000, 1024, 3, 4),
                                        (700, 3, 3, 5)])
def test_permute_bit_exact(T, E, k, seed):
    rng = np.random.default_rng(seed)
    if E <= 128:
        idx = np.stack([rng.permutation(E)[:k] for _ in range(T)]).astype(np.int32)
    else:
        idx = rng.integers(0, E, size=(T, k)).astype(np.int32)
    if seed == 2:
        idx[idx == 7] = 8           # leave an expert empty
    offsets, slot_of, src_of = tq.tq_permute(torch.from_numpy(idx).to(DEV), E)
    torch.cuda.synchronize()
    ro, rs, rsrc = oracle.permute(idx, E)
    assert np.array_equal(offsets.cpu().numpy(), ro)
    assert np.array_equal(slot_of.cpu().numpy(), rs)
    assert np.array_equal(src_of.cpu().numpy(), rsrc)


@pytest.mark.parametrize("T,E,k,S_unused,seed", [(129, 8, 2, 0, 10), (1024, 60, 4, 0, 11), (4096, 64, 6, 0, 12), (4097, 64, 8, 0, 13),
                                                 (2731, 100, 12, 0, 14), (2000, 700, 2, 0, 15), (300, 1024, 1, 0, 16),
                                                 (5000, 1024, 3, 0, 17), (32768, 5, 1, 0, 18), (33, 128, 8, 0, 19),
                                                 (1365, 7, 3, 0, 21), (1366, 7, 3, 0, 22), (2048, 3, 2, 0, 23), (512, 250, 8, 0, 24)])
def test_permute_mid_sized_batches_bit_exact(T, E, k, S_unused, seed):
    """Batches of 257 to 32784 assignments, placed by workgroups of 1024 that count all assignments themselves (up to 4096) or
    add up the counts of a launch of its own: ragged last chunks, empty experts, skewed loads, few and many
    experts, 4095 / 4098 assignments on either side of that limit."""
    print(f"permute T={T} E={E} k={k}", flush=True)
    rng = np.random.default_rng(seed)
    p = rng.random(E) ** 3
    p[rng.integers(0, E)] = 0.0          # one empty expert
    p /= p.sum()
    if k == 1:
        idx = rng.choice(E, size=(T, 1), p=p).astype(np.int32)
    else:
        idx = np.stack([rng.choice(E, size=k, replace=False, p=None if np.count_nonzero(p) < k else p) for _ in range(T)]).astype(np.int32)
    offsets, slot_of, src_of = tq.tq_permute(torch.from_numpy(idx).to(DEV), E)
    torch.cuda.synchronize()
    ro, rs, rsrc = oracle.permute(idx, E)
    assert np.array_equal(offsets.cpu().numpy(), ro)
    assert np.array_equal(slot_of.cpu().numpy(), rs)
    assert np.array_equal(src_of.cpu().numpy(), rsrc)


def test_permute_mid_sized_batch_flags_out_of_range_index():
    rng = np.random.default_rng(20)
    idx = rng.integers(0, 16, size=(1500, 2)).astype(np.int32)
    idx[777, 1] = 16
    idx[3, 0] = -5
    err = torch.zeros(1, dtype=torch.int32, device=DEV)
    offsets, slot_of, src_of = tq.tq_permute(torch.from_numpy(idx).to(DEV), 16, err_flag=err)
    torch.cuda.synchronize()
    assert int(err.item()) & 1
    so = slot_of.cpu().numpy().reshape(1500, 2)
    assert so[777, 1] == -1 and so[3, 0] == -1
    good = idx.copy().reshape(-1)
    keep = (good >= 0) & (good < 16)
    assert int(offsets.cpu().numpy()[-1]) == int(keep.sum())
    # the valid assignments are placed as in a batch without the two bad ones (stable within each expert)
    order = np.argsort(np.where(keep, good, 99), kind="stable")[:keep.sum()]
    assert np.array_equal(src_of.cpu().numpy()[:keep.sum()], order.astype(np.int32))


def test_permute_flags_out_of_range_index():
    idx = np.array([[0, 1], [2, 9], [1, 0]], dtype=np.int32)
    err = torch.zeros(1, dtype=torch.int32, device=DEV)
    offsets, slot_of, src_of = tq.tq_permute(torch.from_numpy(idx).to(DEV), 4, err_flag=err)
    torch.cuda.synchronize()
    assert int(err.item()) & 1
    assert offsets.cpu().numpy().tolist() == [0, 2, 4, 5, 5]
    assert slot_of.cpu().numpy().tolist() == [0, 2, 4, -1, 3, 1]


# ------------------------------------------------------------------ forward
def run_forward(cfg, act, flags=0, bias_override=None):
    layer = get_layer(cfg)
    x = make_x(cfg)
    logits, bias = make_logits(cfg)
    packed = pack_layer_gpu(layer)
    idx, w = tq.tq_route(torch.from_numpy(logits).to(DEV), None if bias is None else torch.from_numpy(bias).to(DEV), cfg.k)
    desc = desc_of(cfg, act, flags)
    ws = torch.empty(tq.tq_moe_workspace_size(desc, cfg.T), dtype=torch.uint8, device=DEV)
    y = tq.tq_moe_forward(desc, packed, x_device(x, act), idx, w, workspace=ws)
    torch.cuda.synchronize()
    assert int(ws[:4].view(torch.int32).item()) == 0
    ridx, rw = oracle.route(logits, bias, cfg.k)
    assert np.array_equal(idx.cpu().numpy(), ridx)
    # the oracle consumes the GPU's own fp32 routing weights: the forward is compared on identical inputs
    ref = oracle.moe_forward_layer(layer, x, ridx, w.cpu().numpy())
    return y.float().cpu().numpy(), ref


@pytest.mark.parametrize("name", list(SMALL))
def test_forward_fp32_debug_path(name):
    got, ref = run_forward(SMALL[name], tq.TQ_ACT_FP32)
    assert rel_err(got, ref) <= TOL_FP32


def test_forward_fp32_config1():
    got, ref = run_forward(CONFIGS[1], tq.TQ_ACT_FP32)
    assert rel_err(got, ref) <= TOL_FP32


@pytest.mark.parametrize("flags", [tq.TQ_FLAG_FORCE_SMALL_TILE, tq.TQ_FLAG_FORCE_LARGE_TILE, tq.TQ_FLAG_FORCE_SKINNY, 0],
                         ids=["tile32", "tile_large", "tile16", "auto"])
@pytest.mark.parametrize("name", list(SMALL))
def test_forward_bf16_small_layers(name, flags):
    got, ref = run_forward(SMALL[name], tq.TQ_ACT_BF16, flags)
    assert rel_err(got, ref) <= TOL_BF16


@pytest.mark.parametrize("flags", [tq.TQ_FLAG_FORCE_SMALL_TILE, tq.TQ_FLAG_FORCE_LARGE_TILE, tq.TQ_FLAG_FORCE_SKINNY],
                         ids=["tile32", "tile_large", "tile16"])
def test_forward_bf16_config1(flags):
    got, ref = run_forward(CONFIGS[1], tq.TQ_ACT_BF16, flags)
    err = rel_err(got, ref)
    print(f"config 1 bf16 flags={flags}: rel err {err:.3e}")
    assert err <= TOL_BF16


@pytest.mark.parametrize("flags", [tq.TQ_FLAG_FORCE_SMALL_TILE, tq.TQ_FLAG_FORCE_LARGE_TILE, tq.TQ_FLAG_FORCE_SKINNY],
                         ids=["tile32", "tile_large", "tile16"])
def test_forward_bf16_is_run_to_run_deterministic(flags):
    cfg = SMALL["ragged"]
    a, _ = run_forward(cfg, tq.TQ_ACT_BF16, flags)
    b, _ = run_forward(cfg, tq.TQ_ACT_BF16, flags)
    assert np.array_equal(a, b)
