// What the tiled kernels read that follows from the blob alone (dense codes: the zero-point fragments that such blobs do not
// store; fp8 factors: fp16 fragments and their placement table), derived into the workspace by workgroups that ride in the
// permutation's launch (tq_route.hip).
#pragma once
#include "tq_device.h"

namespace tqprep {

struct PackGeom {
    int32_t n_exp, H, F, g, r, r16, qmax, cw;
    TqSection gu, d;
    size_t expert_stride;
};

inline PackGeom make_geom(const TqLayout& L)
{
    PackGeom G;
    G.n_exp = L.E + L.S; G.H = L.H; G.F = L.F; G.g = L.g; G.r = L.r; G.r16 = L.r16;
    G.qmax = (1 << L.bits) - 1;
    G.cw = L.cw;
    G.gu = L.gu; G.d = L.d; G.expert_stride = L.expert_stride;
    return G;
}

__device__ inline uint32_t bf16_rne_bits(float f)
{
    uint32_t u = __float_as_uint(f);
    return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}

// bf16 hi (which 0) or lo (which 1) part of c = -scale * (128 + zero), the coefficient of the group sum of the
// activations once the codes are fed to the MFMA as 128 + q; sz = scale | zero << 16 (fp16 bits)
__device__ inline uint32_t zc_part(uint32_t sz, int which)
{
    const float s = __half2float(__ushort_as_half((uint16_t)(sz & 0xFFFF))), z = __half2float(__ushort_as_half((uint16_t)(sz >> 16)));
    const float c = -s * (128.0f + z);
    const uint32_t hi = bf16_rne_bits(c);
    return which == 0 ? hi : bf16_rne_bits(c - __uint_as_float(hi << 16));
}

// fp8 factor fragments of the blob -> fp16 fragments in the workspace, for the tiled kernels (which read fp16
// fragments): left factors with Sigma folded in, A16 = fp16(fp8(A8) * sigma) (one rounding to nearest), right factors
// exactly.  One thread per 8-element fragment of one block; blocks are experts (per-expert factors) or tiles.  A block is a
// whole number of waves, so that block, section and tile are the same over a wave and found by scalar arithmetic.
// which: 0 left factors, 1 right factors.
__device__ inline void expand_fp8(const PackGeom& G, const TqFactorMap& src, const TqFactorMap& dstm, const uint8_t* __restrict__ blob,
                                  uint8_t* __restrict__ fbase, int which, unsigned wave, int lane)
{
    const unsigned n_gu = which == 0 ? (unsigned)G.gu.na_tiles * (G.gu.K / 16) : (unsigned)G.gu.pairs * (G.r16 / 16) * 2;
    const unsigned n_d = which == 0 ? (unsigned)G.d.na_tiles * (G.d.K / 16) : (unsigned)G.d.pairs * (G.r16 / 16) * 2;
    const unsigned per = n_gu + n_d, blk = wave / per;
    unsigned u = wave - blk * per;      // wave inside the section
    const bool is_d = u >= n_gu;
    if (is_d) u -= n_gu;
    const TqSection& sec = is_d ? G.d : G.gu;
    const size_t w = (size_t)u * 64 + lane;
    const uint8_t* sp;        // the block's fp8 fragments
    if (src.shared)
        sp = blob + (which == 0 ? src.apool[is_d] + (size_t)blk * src.astride[is_d]
                                : src.bpool[is_d] + (size_t)blk * src.bstride[is_d]);
    else
        sp = blob + TQ_HEADER_BYTES + (size_t)blk * G.expert_stride + (which == 0 ? sec.afrag : sec.bfrag);
    uint8_t* dp = fbase + (which == 0 ? dstm.apool[is_d] + (size_t)blk * dstm.astride[is_d]
                                      : dstm.bpool[is_d] + (size_t)blk * dstm.bstride[is_d]);
    const uint2 raw = reinterpret_cast<const uint2*>(sp)[w];
    float sg = 1.f;
    if (which == 0) {
        // column of t this fragment belongs to: 32 ta + lane % 32; Sigma is stored per column (gate then up in GU)
        const unsigned ta = u / (unsigned)(sec.K / 16);
        const int c = 32 * (int)ta + (lane & 31), na = is_d ? G.r16 : 2 * G.r16;
        const float* sig = src.shared ? reinterpret_cast<const float*>(blob + src.sig_off[is_d])
                                      : reinterpret_cast<const float*>(blob + TQ_HEADER_BYTES + (size_t)blk * G.expert_stride + sec.sig);
        sg = c < na ? sig[c] : 0.f;
    }
    uint32_t o[4];
#pragma unroll
    for (int i = 0; i < 8; i += 2) {
        const uint32_t b0 = ((i < 4 ? raw.x : raw.y) >> (8 * (i & 3))) & 0xFF, b1 = ((i < 4 ? raw.x : raw.y) >> (8 * ((i + 1) & 3))) & 0xFF;
        const uint32_t h0 = __half_as_ushort(__float2half(tq_fp8_to_float(b0) * sg));
        const uint32_t h1 = __half_as_ushort(__float2half(tq_fp8_to_float(b1) * sg));
        o[i >> 1] = h0 | (h1 << 16);
    }
    reinterpret_cast<uint4*>(dp)[w] = make_uint4(o[0], o[1], o[2], o[3]);
}

// placement table of the expanded factors: the blob's own (shared factors) or the identity (per-expert factors)
__device__ inline void expand_phi(const TqFactorMap& src, const TqFactorMap& dstm, const uint8_t* __restrict__ blob,
                                  uint8_t* __restrict__ fbase, int n_exp, size_t e)
{
    if (e >= (size_t)n_exp) return;
    int32_t* dst = reinterpret_cast<int32_t*>(fbase + dstm.phi_off);
    if (src.shared) {
        const int32_t* p = reinterpret_cast<const int32_t*>(blob + src.phi_off);
        dst[2 * e] = p[2 * e]; dst[2 * e + 1] = p[2 * e + 1];
    } else {
        dst[2 * e] = (int32_t)e; dst[2 * e + 1] = (int32_t)e;
    }
}

// The same zc fragments as packing derives, computed from the blob's own sz part into a buffer outside the blob (dense
// codes on the tiled kernels: such blobs store no zc part).  One thread per (pair, block of 16 groups, tile, lane): it
// reads its 8 scale / zero words once and writes the hi and the lo fragment; all but the lane is the wave's.
__device__ inline void zc_from_blob(const PackGeom& G, const uint8_t* __restrict__ blob, uint8_t* __restrict__ zc_ws,
                                    size_t zc_stride, size_t zc_d_off, unsigned wave, int lane)
{
    const unsigned n_gu = (unsigned)G.gu.pairs * (G.gu.zfrag / 2) * 2;
    const unsigned n_d = (unsigned)G.d.pairs * (G.d.zfrag / 2) * 2;
    const unsigned per = n_gu + n_d, e = wave / per;
    unsigned u = wave - e * per;
    const bool is_d = u >= n_gu;
    if (is_d) u -= n_gu;
    const TqSection& sec = is_d ? G.d : G.gu;
    const int zfrag = sec.zfrag, groups = sec.groups;
    const int tile = (int)(u & 1);
    const unsigned ps = u >> 1, nblocks = (unsigned)zfrag / 2;
    const unsigned pair = ps / nblocks;
    const int gblock = (int)(ps - pair * nblocks);
    const int col = lane & 31, hf = lane >> 5;
    const uint32_t* sz = reinterpret_cast<const uint32_t*>(blob + TQ_HEADER_BYTES + (size_t)e * G.expert_stride + sec.sz);
    uint32_t v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int grp = min(16 * gblock + 8 * hf + i, groups - 1);
        v[i] = sz[(((size_t)pair * groups + grp) * 2 + tile) * 32 + col];
    }
    uint32_t hi[4], lo[4];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const bool live = 16 * gblock + 8 * hf + i < groups;
        const uint32_t h = live ? zc_part(v[i], 0) : 0u, l = live ? zc_part(v[i], 1) : 0u;
        if (i & 1) { hi[i >> 1] |= h << 16; lo[i >> 1] |= l << 16; }
        else { hi[i >> 1] = h; lo[i >> 1] = l; }
    }
    // fragment f of (pair, tile, lane) sits at ((pair * zfrag + f) * 2 + tile) * 64 + lane, 8 values each
    uint4* base = reinterpret_cast<uint4*>(zc_ws + (size_t)e * zc_stride + (is_d ? zc_d_off : 0));
    base[(((size_t)pair * zfrag + 2 * gblock) * 2 + tile) * 64 + lane] = make_uint4(hi[0], hi[1], hi[2], hi[3]);
    base[(((size_t)pair * zfrag + 2 * gblock + 1) * 2 + tile) * 64 + lane] = make_uint4(lo[0], lo[1], lo[2], lo[3]);
}

}  // namespace tqprep

// The parts are independent of the permutation and of each other: consecutive ranges of waves, ending at end[0..3].  Bound by memory and,
// in small layers, by the launch: one of their own took 6 to 12 us between the permutation and the pre-pass, in the permutation's
// launch, whose few workgroups wait for latency, that is hidden.  All indices but the lane are the wave's: indexed per thread, with
// 64-bit divisions and the arguments picked through vector loads, 135 000 waves took 52 us for 207 MB.  Whole call, before and after
// both: 12 experts of 768x2304, 80 tokens, fp8 factors and 3-bit codes 65.4 -> 58.6 us; 8 of 256x512, 120 tokens, fp8 41.2 -> 38.7; 66 of
// 2048x1408, 1531 tokens, both 335 -> 327; 128 of 4096x1536, 300 tokens, fp8 409 -> 401; 200 of 2048x2048, 600 tokens, 2-bit codes
// 355.6 -> 342 (as a launch of its own with the same code: 353).
struct TqPrep {
    tqprep::PackGeom G;
    TqFactorMap src, dstm;
    const uint8_t* blob;
    uint8_t *fbase, *zc_ws;
    size_t zc_stride, zc_d_off;
    unsigned end[4];
    unsigned n_waves;
};

// wave: the same on all lanes
__device__ inline void tq_prep_wave(const TqPrep& P, unsigned wave, int lane)
{
    if (wave < P.end[0]) tqprep::expand_phi(P.src, P.dstm, P.blob, P.fbase, P.G.n_exp, (size_t)wave * 64 + lane);
    else if (wave < P.end[1]) tqprep::expand_fp8(P.G, P.src, P.dstm, P.blob, P.fbase, 0, wave - P.end[0], lane);
    else if (wave < P.end[2]) tqprep::expand_fp8(P.G, P.src, P.dstm, P.blob, P.fbase, 1, wave - P.end[1], lane);
    else if (wave < P.end[3]) tqprep::zc_from_blob(P.G, P.blob, P.zc_ws, P.zc_stride, P.zc_d_off, wave - P.end[2], lane);
}
