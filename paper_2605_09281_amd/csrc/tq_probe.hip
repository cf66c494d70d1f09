// Measurement aid (not part of the method): the instruction mix of the prefill kernels' main loop without any global
// memory traffic, to find what the compute units sustain for it.  One workgroup of four waves per launch slot, each
// wave on a 64 x 64 output tile (2 x 2 MFMA tiles of 32 x 32) walking over groups of 8 steps of 16, as
// moe_prefill_kernel does for quantisation groups of 128:
//   level 0: the MFMAs alone, operands in registers (four independent accumulator chains)
//   level 1: + the two A fragments of every step read from LDS (ds_read_b128)
//   level 2: + the two B fragments of every step unpacked from 4-bit codes (3 shifts and 4 and-or per fragment)
//   level 3: + the fold of every group's partial sums into the accumulators (16 FMAs per tile and group)
//   level 4: + per group, the store of the next activation tile into the other half of an LDS double buffer (four
//            16-byte stores per thread) and the workgroup barrier that publishes it
// Every level runs with two workgroups per compute unit (two waves per SIMD), as the kernel does.  The kernel reports
// its own cycle count and wall-clock time, so the clock the chip sustained under that load is known.
// Operands are random: activations of a normal distribution in bf16, codes of all values (128 + q as bf16 where nothing is unpacked).  The
// chip is at its power limit under such a load; with constant operands, which switch hardly any gate, the same MFMAs run at 2.4 GHz
// and the figures are up to 40 % too good.
#include "tq_device.h"

using namespace tqdev;

namespace {

__device__ inline uint32_t probe_hash(uint32_t v)
{
    v ^= v >> 16; v *= 0x7FEB352Du; v ^= v >> 15; v *= 0x846CA68Bu;
    return v ^ (v >> 16);
}
// two bf16 values of (nearly) a standard normal distribution: the sum of four random bytes, centred
__device__ inline uint32_t probe_normals(uint32_t seed)
{
    uint32_t o = 0;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const uint32_t h = probe_hash(2 * seed + i);
        const float f = ((float)((h & 255) + ((h >> 8) & 255) + ((h >> 16) & 255) + (h >> 24)) - 510.f) * (1.f / 147.8f);
        o |= (__float_as_uint(f) >> 16) << (16 * i);
    }
    return o;
}

template <int LEVEL>
__global__ void __launch_bounds__(256, 2) issue_probe_kernel(float* __restrict__ out, int iters, uint32_t mask, uint32_t magic_s,
                                                             const float* __restrict__ scales,
                                                             unsigned long long* __restrict__ clk)
{
    constexpr int MT = 2, NT = 2, GS = 8, ROWB = 272, BUFB = 32 * MT * ROWB;
    constexpr int NBUF = LEVEL >= 4 ? 2 : 1;
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    for (int i = threadIdx.x; i < (NBUF * BUFB) / 4; i += blockDim.x) reinterpret_cast<uint32_t*>(lds)[i] = probe_normals(i);
    __syncthreads();
    u32x4 xr[MT];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int j = 0; j < 4; ++j) xr[m][j] = probe_normals(0x10000u + (threadIdx.x * MT + m) * 4 + j);
    const uint32_t wr_off = (threadIdx.x >> 4) * ROWB + (threadIdx.x & 15) * 16;      // 16 rows x 256 bytes per pass
    const int lane = threadIdx.x & 63, col = lane & 31, hf = lane >> 5;
    uint32_t magic;
    asm volatile("v_mov_b32 %0, %1" : "=v"(magic) : "s"(magic_s));
    f32x16 acc[MT][NT];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[m][t][v] = 0.f;
    uint32_t w[NT][GS];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int s = 0; s < GS; ++s) w[t][s] = probe_hash(0x20000u + (threadIdx.x * NT + t) * GS + s);
    constexpr int NREG = LEVEL < 2 ? GS : 1;      // register operands: fragments of their own for every step
    Frag areg[NREG][MT], breg[NREG][NT];
#pragma unroll
    for (int s = 0; s < NREG; ++s)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
#pragma unroll
            for (int m = 0; m < MT; ++m) areg[s][m].u[j] = probe_normals(0x30000u + ((threadIdx.x * GS + s) * MT + m) * 4 + j);
#pragma unroll
            for (int t = 0; t < NT; ++t)
                breg[s][t].u[j] = 0x43004300u | (probe_hash(0x50000u + ((threadIdx.x * GS + s) * NT + t) * 4 + j) & 0x000F000Fu);
        }
    const uint8_t* base0 = lds + col * ROWB + hf * 16;
    const unsigned long long c0 = clock64(), w0 = wall_clock64();
    for (int it = 0; it < iters; ++it) {
        float sc[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) sc[t] = scales[(it * NT + t) & 63];
        const uint8_t* base = base0 + (LEVEL >= 4 ? (it & 1) * BUFB : 0);
        f32x16 part[MT][NT];
#pragma unroll
        for (int ks = 0; ks < GS; ++ks) {
            Frag a[MT];
            bf16x8 b[NT];
#pragma unroll
            for (int m = 0; m < MT; ++m) {
                if (LEVEL >= 1) a[m].q = *reinterpret_cast<const u32x4*>(base + m * 32 * ROWB + ((ks + it) & 7) * 32);
                else a[m] = areg[ks % NREG][m];
            }
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                if (LEVEL >= 2) b[t] = unpack_word(w[t][ks] + it, mask, magic);
                else b[t] = breg[ks % NREG][t].v;
            }
#pragma unroll
            for (int m = 0; m < MT; ++m)
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    if (LEVEL >= 3) {
                        if (ks == 0) {
                            f32x16 z;
#pragma unroll
                            for (int v = 0; v < 16; ++v) z[v] = 0.f;
                            part[m][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[m].v, b[t], z, 0, 0, 0);
                        } else {
                            part[m][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[m].v, b[t], part[m][t], 0, 0, 0);
                        }
                    } else {
                        acc[m][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[m].v, b[t], acc[m][t], 0, 0, 0);
                    }
                }
        }
        if (LEVEL >= 3) {
#pragma unroll
            for (int m = 0; m < MT; ++m)
#pragma unroll
                for (int t = 0; t < NT; ++t)
#pragma unroll
                    for (int v = 0; v < 16; ++v) acc[m][t][v] = fmaf(sc[t], part[m][t][v], acc[m][t][v]);
            if (LEVEL >= 4) {
                uint8_t* dst = lds + ((it + 1) & 1) * BUFB + wr_off;
#pragma unroll
                for (int m = 0; m < MT * 2; ++m) *reinterpret_cast<u32x4*>(dst + m * 16 * ROWB) = xr[m % MT];
                lds_barrier();
            }
        } else if (LEVEL < 2) {
            // keep the register operands loop-variant so that the steps are not merged
#pragma unroll
            for (int t = 0; t < NT; ++t) breg[0][t].u[0] ^= (uint32_t)(sc[t] != 7.f);
        }
    }
    const unsigned long long c1 = clock64(), w1 = wall_clock64();
    if (blockIdx.x == 0 && threadIdx.x == 0) { clk[0] = c1 - c0; clk[1] = w1 - w0; }
    float s = 0.f;
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int v = 0; v < 16; ++v) s += acc[m][t][v];
    if (s == 1.2345f) out[threadIdx.x] = s;      // practically never: keeps the result alive
}

}  // namespace

// MFMAs one wave issues per launch: iters groups of 8 steps on 2 x 2 tiles
extern "C" tq_status tq_debug_issue_probe(int32_t level, int32_t iters, void* scratch, size_t scratch_bytes, void* stream)
{
    if (!scratch) return TQ_ERR_NULL;
    if ((uintptr_t)scratch & 255) return TQ_ERR_ALIGN;
    if (level < 0 || level > 4 || iters < 1 || iters > (1 << 20)) return TQ_ERR_SHAPE;
    if (scratch_bytes < 4096) return TQ_ERR_WORKSPACE;
    const TqDeviceState* ds = nullptr;
    if (tqi_device_state(&ds) != TQ_OK) return TQ_ERR_HIP;
    // scratch: [0, 16) the two counters, [256, 512) 64 scales (whatever the caller left there: any finite values),
    // [1024, 2048) the never-written result
    unsigned long long* clk = reinterpret_cast<unsigned long long*>(scratch);
    const float* scales = reinterpret_cast<const float*>(reinterpret_cast<uint8_t*>(scratch) + 256);
    float* out = reinterpret_cast<float*>(reinterpret_cast<uint8_t*>(scratch) + 1024);
    const size_t smem = (level >= 4 ? 2 : 1) * 32 * 2 * 272 + 64;
    const dim3 grid(2 * ds->n_cu), block(256);
    hipStream_t st = (hipStream_t)stream;
    switch (level) {
    case 0: hipLaunchKernelGGL(issue_probe_kernel<0>, grid, block, smem, st, out, iters, 0x000F000Fu, 0x43004300u, scales, clk); break;
    case 1: hipLaunchKernelGGL(issue_probe_kernel<1>, grid, block, smem, st, out, iters, 0x000F000Fu, 0x43004300u, scales, clk); break;
    case 2: hipLaunchKernelGGL(issue_probe_kernel<2>, grid, block, smem, st, out, iters, 0x000F000Fu, 0x43004300u, scales, clk); break;
    case 3: hipLaunchKernelGGL(issue_probe_kernel<3>, grid, block, smem, st, out, iters, 0x000F000Fu, 0x43004300u, scales, clk); break;
    default: hipLaunchKernelGGL(issue_probe_kernel<4>, grid, block, smem, st, out, iters, 0x000F000Fu, 0x43004300u, scales, clk); break;
    }
    TQ_CHECK_LAUNCH();
    return TQ_OK;
}
