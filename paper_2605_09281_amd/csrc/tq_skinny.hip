// Decode path of tq_moe_forward (few rows per expert): the projection is bound by streaming the packed
// weights from HBM once, so the kernel is built around that stream.
//
//   * A row tile holds at most 16 assignment rows of one expert.  Its activations for the whole
//     contraction range of the workgroup (up to 4096 values per row) are staged in LDS ONCE.
//   * A workgroup has 8 waves (2 or 4 on contractions up to 512 or 1024); wave w owns a 512-wide slice (256 on contractions up to 2048) of the contraction range and walks over the
//     workgroup's column-tile pairs, streaming its slice of the packed codes (already in MFMA fragment
//     order) straight from global memory into registers, one pair ahead.  No barrier in that stream.
//   * Codes go to v_mfma_f32_16x16x32_bf16 as 128 + q; each quantisation group's fp32 partial sum is folded as
//     acc += s * part - s (128 + z) * xsum, with the group sums of the activations added up as the rows are staged.  The blob's
//     fragments are those of the 32x32x16 instruction of the tiled kernels; one row exchange (v_permlane16_swap) of the words of
//     two steps makes the 16-column fragments of a 32-deep step of them, so no MFMA row is padding.
//   * The waves' partial results of a pair are summed across the waves through LDS in a fixed order (the
//     "wavefront reduction"), then SwiGLU (stage 0) or the store of the split-K plane (stage 1).
//   * The low-rank intermediate t = x A of a workgroup's range comes as up to four fp32 parts from skinny_pre_kernel (for decode batches
//     proper that of gate/up per assignment from the permutation's launch); a split contraction needs no global reduction: the
//     partial t of a split times B lands in that split's output plane, and the planes are summed by the combine.
// Measured, whole calls (before: 32x32 MFMAs half of whose rows were padding, the intermediate added up from fp32 slices in the set-up,
// group sums by MFMAs against ones, a reduction with a branch per result): 8 experts of 4096 x 14336, 16 tokens 161 -> 145 us, 1 token 67.5 -> 59.7
// (gate/up 32.9 -> 28.1 for 125 MB, down 22.3 -> 17.8 for 63), 16 tokens with codes of 3 bits and fp8 factors 158 -> 134; 128 experts of
// 4096 x 1536, 16 tokens 104 -> 93.
// Tried: two pairs in flight (spills at 512 indices a wave; at 256 the deal gets coarser: 44.6 -> 52.2 us on 60 experts of 2048 x 1408, 4
// tokens); touching every workgroup's first pair in the launch before (down 2 us shorter, that launch 2 us longer).
#include "tq_device.h"

#include <algorithm>
#include <type_traits>

using namespace tqdev;

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

// waves per SIMD that a workgroup of nw waves is compiled for: three where it fits 168 registers without a spill.  (Four, 128 registers: 80
// to 100 bytes spilled and two workgroups per CU, 60 experts of 2048 x 1408, 16 tokens 58.5 -> 72.4 us; two at four waves: 16 experts of 1024 x 8192,
// 8 tokens 47.8 -> 51.8; three at two waves: 24 experts of 512 x 3072, 5 tokens 36.3 -> 37.3.)
constexpr int sk_waves_per_simd(int nw) { return nw == 4 ? 3 : 2; }
constexpr int SK_LDS = 160 * 1024;
// the reduction buffer of NW waves: per wave the 8 - 8 / NW of its results that others add up, 2 tiles, 64 lanes, and a slot for those that nobody reads
constexpr int sk_red_bytes(int nw) { return (nw * (8 - 8 / nw) * 2 + 1) * 64 * 4; }

// Low-rank intermediate of one 16-row tile over 1024 contraction indices (a part of the range of a split):
//   t[tile][split][part][m][c] = sigma_c * sum_{kk in part} x[row m][kk] * A[kk][c]      (fp32)
// One workgroup per (tile, split, part, 32 columns of t); each of its four waves takes a 256-wide slice, with all of its loads in flight
// at once, and the slices are added in order through LDS.  (Left as 256-wide slices for the kernel that reads them, they were 64 loads a lane of its
// set-up.  A whole range of 4096 in one workgroup is 340 KB through one CU, which takes 33 to 50 bytes a ns: 8 experts of 4096 x 14336, 16 tokens
// 7.5 us that way, 5.3 in parts of 1024.)
constexpr int SK_PRE_K = 256;
constexpr int SK_PART_K = TQ_PRE_PART_SLICES * SK_PRE_K;

// Exchanges 16-lane rows: a keeps its even rows and takes b's in its odd ones, b the other way round.  On the words of two 16-deep steps
// (lane = column + 32 * k-half) a becomes the word of a 32-deep step's columns 0..15, b that of columns 16..31; the four rows of either hold
// (step, k-half) = (0, 0), (1, 0), (0, 1), (1, 1).
__device__ inline void swap_rows(uint32_t& a, uint32_t& b)
{
    const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
    a = r[0];
    b = r[1];
}

template <int STAGE, bool FP8>
__global__ void __launch_bounds__(64 * TQ_PRE_PART_SLICES) skinny_pre_kernel(MGeom G, TqSection sec, const uint8_t* __restrict__ blob,
                                                          const uint16_t* __restrict__ xin,
                                                          const int32_t* __restrict__ row_token,
                                                          const int32_t* __restrict__ tile_e,
                                                          const int32_t* __restrict__ tile_row0,
                                                          const int32_t* __restrict__ tile_rows,
                                                          const int32_t* __restrict__ ctrl, float* __restrict__ t_out, int range_k,
                                                          int n_parts)
{
    constexpr int NW = TQ_PRE_PART_SLICES;
    __shared__ float red[NW][8][64];
    const int tile = blockIdx.x, split = blockIdx.y / n_parts, part = blockIdx.y % n_parts, ta = blockIdx.z, lane = threadIdx.x & 63,
              slice = threadIdx.x >> 6;
    if (tile >= ctrl[4]) return;
    const int e = tile_e[tile], slot0 = tile_row0[tile], rows = tile_rows[tile];
    const int K = sec.K, ksteps = K / 16;
    const int r = min(lane & 15, rows - 1), lrow = lane >> 4;
    const uint16_t* xrow = (STAGE == 0 ? xin + (size_t)row_token[slot0 + r] * K : xin + (size_t)(slot0 + r) * K) + 16 * (lrow & 1) + 8 * (lrow >> 1);
    const u32x4* af = reinterpret_cast<const u32x4*>(tq_afrag_base(blob, G.expert_stride, sec, G.fm, STAGE, e)) + (FP8 ? lane >> 1 : lane);
    constexpr int NS = SK_PRE_K / 16;
    const int s0 = split * (range_k / 16) + (part * NW + slice) * NS;
    const int n = min(NS, min(ksteps, (split + 1) * (range_k / 16)) - s0);      // (<= 0: past the end of the last split); even: ranges are whole chunks of 64
    Frag xa[NS / 2];
    u32x4 aq[NS];
#pragma unroll
    for (int u = 0; u < NS; ++u)
        if (u < n) {
            if (u % 2 == 0) xa[u / 2].q = *reinterpret_cast<const u32x4*>(xrow + 16 * (s0 + u));
            const size_t f = (size_t)ta * ksteps + s0 + u;                  // fragment; fp8 fragments are half as long
            aq[u] = af[f * (FP8 ? 32 : 64)];
        }
    f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
    for (int u = 0; u < NS; u += 2)
        if (u < n) {
            Frag b[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) b[i].v = FP8 ? fp8_frag_to_bf8(aq[u + i], lane) : half8_to_bf8(aq[u + i]);
#pragma unroll
            for (int j = 0; j < 4; ++j) swap_rows(b[0].u[j], b[1].u[j]);
#pragma unroll
            for (int i = 0; i < 2; ++i) acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xa[u / 2].v, b[i].v, acc[i], 0, 0, 0);
        }
#pragma unroll
    for (int v = 0; v < 8; ++v) red[slice][v][lane] = acc[v >> 2][v & 3];
    __syncthreads();
    const int NA = STAGE == 0 ? 2 * G.r16 : G.r16;
    for (int i = threadIdx.x; i < 512; i += 64 * NW) {
        const int v = i >> 6, l = i & 63, c = 32 * ta + 16 * (v >> 2) + (l & 15), m = 4 * (l >> 4) + (v & 3);
        if (c >= NA) continue;
        float t = red[0][v][l];
#pragma unroll
        for (int sl = 1; sl < NW; ++sl) t += red[sl][v][l];
        if (FP8) t *= tq_sig_base(blob, G.expert_stride, sec, G.fm, STAGE, e)[c];
        t_out[(((size_t)tile * gridDim.y + blockIdx.y) * 16 + m) * NA + c] = t;
    }
}

// A buffer descriptor of `bytes` bytes at p: loads past its end return zeros without a request, so a load that has nothing to
// fetch (no further pair, a wave without a slice) is switched off by a length of 0 instead of a condition, after which the
// compiler would wait for all loads in flight.
__device__ inline __amdgpu_buffer_rsrc_t buffer(const uint8_t* p, uint32_t bytes)
{
    const uint64_t a = reinterpret_cast<uint64_t>(p);
    const uint64_t u = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)a) |
                       (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(a >> 32)) << 32;
    return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(u), 0, (int)bytes, 0x00020000);
}
constexpr int BUF_NT = 2;      // non-temporal: read once, never again; the hint keeps the stream out of the caches

template <int CTRL>
__device__ inline float dpp_add(float v)
{
    return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}

// the sum of 8 bf16 values a lane over runs of LANES lanes (4, 8, 16 or 32), in every lane of the run
template <int LANES>
__device__ inline float run_sum(const u32x4& q)
{
    float s = ((bf_lo(q[0]) + bf_hi(q[0])) + (bf_lo(q[1]) + bf_hi(q[1]))) + ((bf_lo(q[2]) + bf_hi(q[2])) + (bf_lo(q[3]) + bf_hi(q[3])));
    s = dpp_add<0xB1>(s);                        // lanes 1, 0, 3, 2 of a quad
    s = dpp_add<0x4E>(s);                        // lanes 2, 3, 0, 1
    if (LANES >= 8) s = dpp_add<0x141>(s);       // the row's halves mirrored
    if (LANES >= 16) s = dpp_add<0x140>(s);      // the row mirrored
    if (LANES >= 32) s += __shfl_xor(s, 16);
    return s;
}

// STAGE 0: out = h[slot][F] bf16 = silu(gate) * up.   STAGE 1: out = yd[split][slot][H] fp32.
// CW: 32-bit words of codes per lane, tile and 64-wide chunk: 4 (4-bit slots), 3 or 2 (dense 3- / 2-bit codes).
// WK, NW: contraction indices per wave and waves per workgroup: 512 and 8; on contractions of at most 2048 256 and as many waves
// as they take (2, 4 or 8), and a CU holds as many workgroups as it has room for.
template <int STAGE, int GS, int CW, int WK, int NW>
__global__ void __launch_bounds__(64 * NW, sk_waves_per_simd(NW)) moe_skinny_kernel(MGeom G, TqSection sec, const uint8_t* __restrict__ blob,
                                                         const uint16_t* __restrict__ xin,
                                                         const int32_t* __restrict__ row_token,
                                                         const int32_t* __restrict__ tile_e,
                                                         const int32_t* __restrict__ tile_row0,
                                                         const int32_t* __restrict__ tile_rows,
                                                         const int32_t* __restrict__ ctrl,
                                                         const float* __restrict__ t_in, int n_parts,
                                                         void* __restrict__ out, int32_t* __restrict__ pair_cnt,
                                                         int units_per_split, int RB, int red_off, int xs_off, int mb_off,
                                                         const int32_t* __restrict__ row_src, int nsplit)
{
    constexpr int UNIT_K = (GS * 16 < 64) ? 64 : GS * 16;
    constexpr int UC = UNIT_K / 64;
    constexpr int US = UNIT_K / 32;    // 32-deep MFMA steps per unit
    constexpr int NG = UNIT_K / (GS * 16);
    constexpr int GT = GS / 2;         // steps per group
    constexpr int UPW = WK / UNIT_K;   // units per wave
    constexpr int NT = 64 * NW;
    constexpr int OV = 8 / NW;         // results per tile that a wave adds up, and low-rank steps that it may have
    constexpr int MAXP = NW == 8 ? TQ_PRE_MAX_PARTS : 1;      // parts of the low-rank intermediate (fewer waves: at most 1024 indices)
    using WT = std::conditional_t<CW == 4, u32x4, uint32_t>;      // register type of the packed codes
    constexpr int WN = CW == 4 ? UC : UC * CW;                    // and how many of them one tile of a unit takes
    // dense codes in units of two chunks: a 32-deep step takes step w of both chunks, so that the rows of the raw words can be exchanged
    constexpr bool PAIRED = CW != 4 && UC > 1;

    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    float* red = reinterpret_cast<float*>(lds + red_off);
    float* xs = reinterpret_cast<float*>(lds + xs_off);

    // Which (row tile, split) this workgroup works on, its number `part` among the g_wg workgroups on it: the workgroups are shared out among the
    // combinations that EXIST, a number only the device knows (most experts of a large layer receive no row, hot ones fill several tiles).  Each
    // of the n_v combinations gets G_lo = grid / n_v consecutive workgroups, the first grid mod n_v one more from the end: consecutive ids
    // sit on different XCDs, so a combination's weight stream is spread over all of them.  (A grid sized by the host for one tile
    // an expert runs the tiles beyond in a second round and leaves the experts without rows idle: 8 experts of 4096 x 14336, 48 tokens 237 us against 183 here,
    // 4 tokens 118 against 102; 32 of 2048 x 2048, top-4, 80 tokens 100 against 73; where every expert has one tile the two are level, up to 2 % apart
    // either way.  With combination b mod n_v for workgroup b, 16 tokens of the first layer take 3 % longer: each XCD then streams one expert.)
    int rt, split, part, g_wg;
    {
        const int n_t = ctrl[4], n_v = n_t * nsplit;
        if (n_v == 0) return;
        const unsigned gx = gridDim.x, b = blockIdx.x, G_lo = gx / (unsigned)n_v, n_full = G_lo * (unsigned)n_v;      // the grid has at least n_v workgroups
        const bool extra = b >= n_full;
        const unsigned vq = b / G_lo;
        const int vt = (int)(extra ? b - n_full : vq);
        part = (int)(extra ? G_lo : b - vq * G_lo);
        if (part >= sec.pairs) return;      // more workgroups on this combination than it has pairs
        g_wg = (int)G_lo + (vt < (int)(gx - n_full) ? 1 : 0);
        rt = vt;
        split = 0;
        if (nsplit > 1) {
            split = (int)((unsigned)vt / (unsigned)n_t);
            rt = vt - split * n_t;
        }
    }
    const int e = tile_e[rt], slot0 = tile_row0[rt], rows = tile_rows[rt];
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, col = lane & 31;
    const int l16 = lane & 15, lrow = lane >> 4;      // MFMA: row of A / column of B and D; quarter of the contraction step / of the rows of D
    const int K = sec.K, NU = K / UNIT_K;
    const int NA = STAGE == 0 ? 2 * G.r16 : G.r16;
    const int n_lr = (G.r > 0) ? NA / 16 : 0;       // low-rank MFMA steps; step j is applied by wave j % NW
    const int ub = split * units_per_split;
    const int ue = min(NU, ub + units_per_split);
    const int range_k = (ue - ub) * UNIT_K;
    int nuw = min(UPW, ue - (ub + wave * UPW));     // units of this wave (0 for idle waves)
    if (nuw < 0) nuw = 0;
    // Column-tile pairs are dealt out dynamically among the g_wg workgroups of this (tile, split): the first one is the
    // workgroup's number among them, every further one comes from a counter (cleared by the permutation), fetched one pair
    // before its weights are requested.  Workgroups that get a better share of the
    // memory system take more pairs, and all of them finish together.
    const int npairs = sec.pairs;
    int32_t* cnt = pair_cnt + (size_t)rt * TQ_MAX_SPLIT + split;
    int* pq = reinterpret_cast<int*>(lds + mb_off);            // two mailbox words, in turn
    int got_v = 0;
    if (tid == 0) got_v = g_wg + atomicAdd(cnt, 1);

    const uint8_t* rec = blob + TQ_HEADER_BYTES + (size_t)e * G.expert_stride;
    const bool fp8 = G.fm.fp8 != 0;
    // fragment f of the right factors: 64 lanes x 16 bytes (fp16), or 64 x 8 bytes (fp8: lanes 2j, 2j + 1 share a word)
    const int b_per = fp8 ? 512 : 1024, b_lane = (fp8 ? (lane >> 1) : lane) * 16;
    const uint8_t* bfr = G.r > 0 ? tq_bfrag_base(blob, G.expert_stride, sec, G.fm, STAGE, e) : rec;
    const uint32_t codes_bytes = (uint32_t)sec.pairs * sec.chunks * (512 * CW), sz_bytes = (uint32_t)sec.pairs * sec.groups * 256;
    const int steps_per_tile = G.r16 / 16;
    const uint32_t b_bytes = (uint32_t)sec.pairs * steps_per_tile * 2 * b_per;

    auto load_w = [&](WT (&dst)[2][WN], int pair, int u) {       // unit u of this wave, both tiles
        const __amdgpu_buffer_rsrc_t rs = buffer(rec + sec.codes, pair < npairs && u < nuw ? codes_bytes : 0u);
        const int so = (pair * sec.chunks + (ub + wave * UPW + u) * UC) * (512 * CW);
        int lo = lane * (CW == 4 ? 16 : 4);
        asm volatile("" : "+v"(lo));      // one register; the rest of the offset goes into the instruction
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int c = 0; c < UC; ++c) {
                if constexpr (CW == 4) {
                    dst[t][c] = __builtin_amdgcn_raw_buffer_load_b128(rs, lo + (c * 2 + t) * 1024, so, BUF_NT);
                } else {
#pragma unroll
                    for (int d = 0; d < CW; ++d)
                        dst[t][c * CW + d] = __builtin_amdgcn_raw_buffer_load_b32(rs, lo + ((c * 2 + t) * CW + d) * 256, so, BUF_NT);
                }
            }
    };
    auto load_sz = [&](uint32_t (&dst)[NG][2], int pair, int u) {
        const __amdgpu_buffer_rsrc_t rs = buffer(rec + sec.sz, pair < npairs && u < nuw ? sz_bytes : 0u);
        const int so = (pair * sec.groups + (ub + wave * UPW + u) * NG) * 256;
#pragma unroll
        for (int gi = 0; gi < NG; ++gi)
#pragma unroll
            for (int t = 0; t < 2; ++t) dst[gi][t] = __builtin_amdgcn_raw_buffer_load_b32(rs, col * 4 + (gi * 2 + t) * 128, so, 0);
    };
    // low-rank B fragments ride in the same prefetch: steps wave, wave + NW, ... (stage 0: steps below r16 / 16 feed the gate tile, the others the up tile)
    constexpr int NBQ = STAGE == 0 ? 1 : 2;
    auto load_b = [&](u32x4 (&dst)[OV][NBQ], int pair) {
#pragma unroll
        for (int q = 0; q < OV; ++q) {
            const int step = wave + NW * q, t0 = STAGE == 0 && step >= steps_per_tile ? 1 : 0;
            const __amdgpu_buffer_rsrc_t rs = buffer(bfr, pair < npairs && step < n_lr ? b_bytes : 0u);
            const int so = (pair * steps_per_tile + step - t0 * steps_per_tile) * 2 * b_per;
#pragma unroll
            for (int t = 0; t < NBQ; ++t) dst[q][t] = __builtin_amdgcn_raw_buffer_load_b128(rs, b_lane, so + (t0 + t) * b_per, 0);
        }
    };

    // the or-operand of the unpack in a vector register (see unpack_word): opaque move, not folded to a literal
    uint32_t magic_v;
    asm volatile("v_mov_b32 %0, %1" : "=v"(magic_v) : "s"(G.unpack_magic));

    // ---- 1. activations of the tile for the workgroup's contraction range -> LDS (row stride RB = 2*range + 16 bytes:
    //         the rows read by one ds_read_b128 fall into different bank groups), their group sums beside them.  Only the rows that exist are
    //         staged; the MFMA rows beyond them re-read the last one and their results are never stored.
    //         Up to eight rows of 4096 are requested at once, and before the first weights: at kernel start every workgroup asks for its
    //         first pair at once, and small loads queued behind that burst would arrive only after it.  What the set-up waits for is kept
    //         short (the intermediate comes summed up, the group sums cost no loads): it is 6 us of a kernel in which nothing streams.
    const int gran = range_k / 8;                 // 16-byte chunks per row
    const int total = rows * gran;
    auto stage_load = [&](int c0, u32x4 (&v)[4]) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int c = min(c0 + j * NT + tid, total - 1);
            const int row = c / gran, kg = c - row * gran;
            const size_t src_row = STAGE == 0 ? (size_t)row_token[slot0 + row] : (size_t)(slot0 + row);
            v[j] = *reinterpret_cast<const u32x4*>(xin + src_row * K + (size_t)ub * UNIT_K + (size_t)kg * 8);
        }
    };
    auto stage_store = [&](int c0, const u32x4 (&v)[4]) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            // a group is a run of 2 GS chunks (4 to 32, a divisor of 64) and `total` a whole number of them: its lanes are all in range or all not
            const float s = run_sum<2 * GS>(v[j]);
            const int c = c0 + j * NT + tid;
            if (c < total) {
                const int row = c / gran, kg = c - row * gran;
                *reinterpret_cast<u32x4*>(lds + row * RB + kg * 16) = v[j];
                if ((kg & (2 * GS - 1)) == 0) xs[kg / (2 * GS) * 16 + row] = s;
            }
        }
    };
    u32x4 xa0[4], xa1[4];
    const bool two = total > 4 * NT;
    stage_load(0, xa0);
    if (two) stage_load(4 * NT, xa1);
    // ---- low-rank intermediate: the parts of the A operands of this wave's 16-deep steps, rows of a step at lane rows 0 and 2 (the others
    //      meet zeros).  Only what exists, by the waves that have a step: requests in front of the weights are what the set-up waits for
    f32x4 tp[OV][MAXP][2];
    if (wave < n_lr) {
        const bool by_assign = STAGE == 0 && row_src;
        const size_t row = by_assign ? (size_t)row_src[slot0 + min(l16, rows - 1)] * n_parts * NA : (((size_t)rt * nsplit + split) * n_parts * 16 + l16) * NA;
        const float* tr = t_in + row + 16 * wave + 4 * (lrow & 2);
#pragma unroll
        for (int q = 0; q < OV; ++q)
            if (wave + NW * q < n_lr) {
#pragma unroll
                for (int p = 0; p < MAXP; ++p)
                    if (p < n_parts) {
                        const f32x4* src = reinterpret_cast<const f32x4*>(tr + 16 * NW * q + (size_t)p * (by_assign ? NA : 16 * NA));
                        tp[q][p][0] = src[0];
                        tp[q][p][1] = src[1];
                    }
            }
    }
    WT wq[UPW][2][WN];
    uint32_t szq[UPW][NG][2];
    u32x4 bq[OV][NBQ];
#pragma unroll
    for (int u = 0; u < UPW; ++u) { load_w(wq[u], part, u); load_sz(szq[u], part, u); }
    load_b(bq, part);
    stage_store(0, xa0);
    if (two) {
        stage_store(4 * NT, xa1);
        for (int c0 = 8 * NT; c0 < total; c0 += 4 * NT) {      // the rare tall tiles
            stage_load(c0, xa0);
            stage_store(c0, xa0);
        }
    }
    if (tid == 0) pq[0] = got_v;
    lds_barrier();
    Frag tf[OV];
#pragma unroll
    for (int q = 0; q < OV; ++q) {
#pragma unroll
        for (int j = 0; j < 4; ++j) tf[q].u[j] = 0;
        if (wave + NW * q < n_lr) {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                f32x4 t = tp[q][0][i];
#pragma unroll
                for (int p = 1; p < MAXP; ++p)
                    if (p < n_parts) t += tp[q][p][i];
                if ((lrow & 1) == 0) {
                    tf[q].u[2 * i] = pack_bf2(t[0], t[1]);
                    tf[q].u[2 * i + 1] = pack_bf2(t[2], t[3]);
                }
            }
        }
    }
    const int xrow_off = min(l16, rows - 1) * RB + (PAIRED ? 64 * (lrow & 1) + 8 * (lrow >> 1) : 16 * (lrow & 1) + 8 * (lrow >> 1)) * 2 +
                         wave * WK * 2;
    auto lds_x = [&](int s) -> bf16x8 {       // A operand of step s of this wave (a constant at every call)
        const int k = PAIRED ? 128 * (s / 4) + 16 * (s % 4) : 32 * s;
        Frag f;
        f.q = *reinterpret_cast<const u32x4*>(lds + xrow_off + k * 2);
        return f.v;
    };
    auto b_operand = [&](const u32x4& raw, Frag& lo, Frag& hi) {
        lo.v = fp8 ? fp8_frag_to_bf8(raw, lane) : half8_to_bf8(raw);
#pragma unroll
        for (int j = 0; j < 4; ++j) { hi.u[j] = 0; swap_rows(lo.u[j], hi.u[j]); }
    };

    // ---- 2. the stream over this workgroup's column-tile pairs
    int pnext = __builtin_amdgcn_readfirstlane(pq[0]), it = 0;
    for (int pair = part; pair < npairs;) {
        int fetched = 0;
        if (tid == 0) fetched = g_wg + atomicAdd(cnt, 1);       // the pair after the next one
        f32x4 acc[2][2];
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int n = 0; n < 2; ++n) acc[t][n] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int u = 0; u < UPW; ++u) {
            WT wc[2][WN];
            uint32_t szc[NG][2];
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int c = 0; c < WN; ++c) wc[t][c] = wq[u][t][c];
#pragma unroll
            for (int gi = 0; gi < NG; ++gi)
#pragma unroll
                for (int t = 0; t < 2; ++t) szc[gi][t] = szq[u][gi][t];
            load_w(wq[u], pnext, u);
            load_sz(szq[u], pnext, u);
            if (u < nuw) {
                if constexpr (PAIRED) {
#pragma unroll
                    for (int t = 0; t < 2; ++t)
#pragma unroll
                        for (int c = 0; c < UC; c += 2)
#pragma unroll
                            for (int i = 0; i < CW; ++i) swap_rows(wc[t][c * CW + i], wc[t][(c + 1) * CW + i]);
                }
                bf16x8 xq[2];
                xq[0] = lds_x(u * US);
#pragma unroll
                for (int gi = 0; gi < NG; ++gi) {
                    f32x4 pt[2][2];
#pragma unroll
                    for (int ks = 0; ks < GT; ++ks) {
                        const int s = gi * GT + ks;
                        if (s + 1 < US) xq[(s + 1) & 1] = lds_x(u * US + s + 1);   // next step's operand
                        const bf16x8 xa = xq[s & 1];
#pragma unroll
                        for (int t = 0; t < 2; ++t) {
                            Frag bw[2];      // columns 0..15 and 16..31 of the tile
                            if constexpr (CW == 4) {
                                uint32_t w0 = word_of(wc[t][s / 2], 2 * s % 4), w1 = word_of(wc[t][s / 2], 2 * s % 4 + 1);
                                swap_rows(w0, w1);
                                bw[0].v = unpack_word(w0, G.unpack_mask, magic_v);
                                bw[1].v = unpack_word(w1, G.unpack_mask, magic_v);
                            } else if constexpr (PAIRED) {
#pragma unroll
                                for (int n = 0; n < 2; ++n)
                                    bw[n].v = unpack_dense<CW>(&wc[t][(s / 4 * 2 + n) * CW], s % 4, G.unpack_mask, magic_v);
                            } else {
#pragma unroll
                                for (int n = 0; n < 2; ++n)
                                    bw[n].v = unpack_dense<CW>(&wc[t][s / 2 * CW], 2 * (s % 2) + n, G.unpack_mask, magic_v);
#pragma unroll
                                for (int j = 0; j < 4; ++j) swap_rows(bw[0].u[j], bw[1].u[j]);
                            }
#pragma unroll
                            for (int n = 0; n < 2; ++n)
                                pt[t][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xa, bw[n].v, ks == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : pt[t][n],
                                                                                   0, 0, 0);
                        }
                    }
                    // fold the group: acc += s * part + c * xsum, c = -s (128 + z)
                    const int gl = (wave * UPW + u) * NG + gi;
                    const f32x4 xv = *reinterpret_cast<const f32x4*>(xs + gl * 16 + 4 * lrow);
#pragma unroll
                    for (int t = 0; t < 2; ++t) {
                        const float s = tq_half_bits_to_float((uint16_t)(szc[gi][t] & 0xFFFF));
                        const float z = tq_half_bits_to_float((uint16_t)(szc[gi][t] >> 16));
                        const float c = -s * (128.0f + z);
                        // this lane's column is lane % 32; what the two halves of the tile need is that of lane % 16 and of lane % 16 + 16
                        uint32_t sn[2], cn[2];
                        sn[0] = sn[1] = __float_as_uint(s);
                        cn[0] = cn[1] = __float_as_uint(c);
                        swap_rows(sn[0], sn[1]);
                        swap_rows(cn[0], cn[1]);
#pragma unroll
                        for (int n = 0; n < 2; ++n)
#pragma unroll
                            for (int v = 0; v < 4; ++v)
                                acc[t][n][v] = fmaf(__uint_as_float(cn[n]), xv[v], fmaf(__uint_as_float(sn[n]), pt[t][n][v], acc[t][n][v]));
                    }
                }
            }
        }
        {
            u32x4 bc[OV][NBQ];
#pragma unroll
            for (int q = 0; q < OV; ++q)
#pragma unroll
                for (int t = 0; t < NBQ; ++t) bc[q][t] = bq[q][t];
            load_b(bq, pnext);
#pragma unroll
            for (int q = 0; q < OV; ++q)
                if (wave + NW * q < n_lr) {
                    const bool up = STAGE == 0 && wave + NW * q >= steps_per_tile;
#pragma unroll
                    for (int t = 0; t < NBQ; ++t) {
                        Frag lo, hi;
                        b_operand(bc[q][t], lo, hi);
                        if (up) {
                            acc[1][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(tf[q].v, lo.v, acc[1][0], 0, 0, 0);
                            acc[1][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(tf[q].v, hi.v, acc[1][1], 0, 0, 0);
                        } else {
                            acc[t][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(tf[q].v, lo.v, acc[t][0], 0, 0, 0);
                            acc[t][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(tf[q].v, hi.v, acc[t][1], 0, 0, 0);
                        }
                    }
                }
        }
        // ---- wavefront reduction: of the 8 results (half v / 4 of a tile's columns, row v % 4 of each four) wave w adds up OV w, OV w + 1, ...
        //      and publishes the others.  Without branches, so that all reads are under way together: a wave's own results go to a slot that
        //      nobody reads, and in the sum they take the place of what is read for them (with a branch per result and per wave, the reads one
        //      after the other: 8 experts of 4096 x 14336, 4 tokens 128 -> 118 us a call; 128 of 4096 x 1536, 16 tokens 104.4 -> 98.5).
        {
            float* mine = red + wave * ((8 - OV) * 2 * 64) + lane;
            float* none = red + NW * (8 - OV) * 2 * 64 + lane;
#pragma unroll
            for (int v = 0; v < 8; ++v) {
                const bool own = v / OV == wave;
                const int slot = v / OV < wave ? v : v - OV;
#pragma unroll
                for (int t = 0; t < 2; ++t) *(own ? none : mine + (t * (8 - OV) + slot) * 64) = acc[t][v >> 2][v & 3];
            }
            if (tid == 0) pq[(it + 1) & 1] = fetched;
        }
        lds_barrier();
        {
            float part[NW][OV][2], tot[OV][2];
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                const float* src = red + w * ((8 - OV) * 2 * 64) + OV * (wave < w ? wave : max(wave - 1, 0)) * 64 + lane;
#pragma unroll
                for (int i = 0; i < OV; ++i)
#pragma unroll
                    for (int t = 0; t < 2; ++t) part[w][i][t] = src[(t * (8 - OV) + i) * 64];
            }
#pragma unroll
            for (int i = 0; i < OV; ++i)
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    float own = acc[t][i >> 2][i & 3];
#pragma unroll
                    for (int w = 1; w < NW; ++w) own = w == wave ? acc[t][(OV * w + i) >> 2][(OV * w + i) & 3] : own;
                    tot[i][t] = 0.f;
#pragma unroll
                    for (int w = 0; w < NW; ++w) tot[i][t] += w == wave ? own : part[w][i][t];      // fixed order: run-to-run identical sums
                }
#pragma unroll
            for (int i = 0; i < OV; ++i) {
                const int v = OV * wave + i, m = 4 * lrow + (v & 3), n = 16 * (v >> 2) + l16;
                if (m < rows) {
                    if (STAGE == 0) {
                        const float hv = silu_mul(tot[i][0], tot[i][1]);
                        reinterpret_cast<uint16_t*>(out)[(size_t)(slot0 + m) * G.F + 32 * pair + n] = (uint16_t)f2bf_bits(hv);
                    } else {
                        float* yd = reinterpret_cast<float*>(out) + (size_t)split * G.a_tot * G.H + (size_t)(slot0 + m) * G.H + 64 * pair + n;
                        yd[0] = tot[i][0];
                        yd[32] = tot[i][1];
                    }
                }
            }
        }
        lds_barrier();
        pair = pnext;
        pnext = __builtin_amdgcn_readfirstlane(pq[(it + 1) & 1]);
        ++it;
    }
}

template <int STAGE, int GS, int CW, int WK, int NW>
tq_status launch_skinny(const MGeom& G, const TqSection& sec, const uint8_t* blob, const uint16_t* xin,
                        const int32_t* row_token, const int32_t* tile_e, const int32_t* tile_row0,
                        const int32_t* tile_rows, const int32_t* ctrl, const float* t_in, int n_parts,
                        void* out, int32_t* pair_cnt, int row_tiles, int nsplit, int units_per_split,
                        hipStream_t st, const int32_t* row_src)
{
    constexpr int UNIT_K = (GS * 16 < 64) ? 64 : GS * 16;
    const int range_k = units_per_split * UNIT_K;
    const int RB = range_k * 2 + 16;
    const int red_off = 16 * RB;
    const int xs_off = red_off + sk_red_bytes(NW);
    const int mb_off = xs_off + (range_k / G.g) * 16 * 4;      // mailbox of the pair scheduler
    const size_t smem = (size_t)mb_off + 16;
    if (smem > SK_LDS) return TQ_ERR_UNSUPPORTED;
    // as many workgroups as the chip holds at once (more, shorter ones would spend more of their time on the set-up: activation staging,
    // group sums)
    const TqDeviceState* ds = nullptr;
    if (tqi_device_state(&ds) != TQ_OK) return TQ_ERR_HIP;
    const long slots = (long)ds->n_cu * std::max<long>(1, std::min<long>(4 * sk_waves_per_simd(NW) / NW, SK_LDS / (long)smem));      // workgroups that the chip holds at once
    // at least one workgroup per (tile, split) that may exist; the kernel shares them out among those that do.  (The dynamic-LDS limit is raised once
    // per device by tqi_setup_skinny.)
    // A combination has work for at most `pairs` of them: small layers launch no more (1024 instead of 160, most of which end at once, cost 8 experts
    // of 256 x 512, 16 tokens, 2 us of 27).
    const long combos = (long)std::min<int64_t>(row_tiles, G.a_tot) * nsplit;
    const long n_wg = std::max<long>(std::min<long>(slots, combos * sec.pairs), (long)row_tiles * nsplit);
    if (n_wg > 0x7FFFFFFF) return TQ_ERR_UNSUPPORTED;
    hipLaunchKernelGGL((moe_skinny_kernel<STAGE, GS, CW, WK, NW>), dim3((unsigned)n_wg), dim3(64 * NW), smem, st, G, sec, blob, xin, row_token, tile_e,
                       tile_row0, tile_rows, ctrl, t_in, n_parts, out, pair_cnt, units_per_split, RB, red_off, xs_off, mb_off, row_src, nsplit);
    TQ_CHECK_LAUNCH();
    return TQ_OK;
}

template <int STAGE>
tq_status launch_skinny_gs(int gs, int cw, const MGeom& G, const TqSection& sec, const uint8_t* blob, const uint16_t* xin,
                           const int32_t* row_token, const int32_t* tile_e, const int32_t* tile_row0,
                           const int32_t* tile_rows, const int32_t* ctrl, const float* t_in, int n_parts,
                           void* out, int32_t* pair_cnt, int row_tiles, int nsplit, int units_per_split,
                           hipStream_t st, const int32_t* row_src, int wave_k, int n_waves)
{
#define TQ_SKL(GSV, CWV, WKV, NWV)                                                                                        \
    return launch_skinny<STAGE, GSV, CWV, WKV, NWV>(G, sec, blob, xin, row_token, tile_e, tile_row0, tile_rows, ctrl, t_in, \
                                                    n_parts, out, pair_cnt, row_tiles, nsplit, units_per_split, st, row_src)
#define TQ_SK(GSV, CWV)                                                                                                   \
    do {                                                                                                                  \
        if (wave_k == 512) TQ_SKL(GSV, CWV, 512, 8);                                                                      \
        if (n_waves == 2) TQ_SKL(GSV, CWV, 256, 2);                                                                       \
        if (n_waves == 4) TQ_SKL(GSV, CWV, 256, 4);                                                                       \
        TQ_SKL(GSV, CWV, 256, 8);                                                                                         \
    } while (0)
    if (cw == 4) {
        switch (gs) {
            case 2: TQ_SK(2, 4);
            case 4: TQ_SK(4, 4);
            case 8: TQ_SK(8, 4);
            case 16: TQ_SK(16, 4);
        }
    } else if (cw == 3) {      // dense codes: groups of 64 and 128
        if (gs == 4) TQ_SK(4, 3);
        if (gs == 8) TQ_SK(8, 3);
    } else if (cw == 2) {
        if (gs == 4) TQ_SK(4, 2);
        if (gs == 8) TQ_SK(8, 2);
    }
#undef TQ_SK
#undef TQ_SKL
    return TQ_ERR_UNSUPPORTED;
}

// Contraction indices per wave of a stage: 512, or 256 on contractions of at most 2048 (with 512 a contraction of 1536 would leave five of
// eight waves idle); waves per workgroup: as many as have a slice (2, 4 or 8).  Eight waves of which four have work keep 32 KB of codes in flight
// per CU, three workgroups of four 96 KB: 16 experts of 1024 x 8192, rank 0, 8 tokens 71.4 -> 47.8 us a call, 30 tokens 77.5 -> 61.5; 32 of 768 x 3072,
// 60 tokens 61.4 -> 46.4; two waves: 24 of 512 x 3072, 5 tokens 42.1 -> 36.3.
inline int wave_k_of(int K, int g) { return (K <= 2048 && g <= 256) ? 256 : 512; }
inline int waves_of(int K, int g) { return wave_k_of(K, g) == 512 || K > 1024 ? 8 : K > 512 ? 4 : 2; }

// contraction split of one stage: nsplit workgroups along K, each a whole number of wave slices
inline void plan_split(int K, int g, int* nsplit, int* units_per_split)
{
    const int unit_k = g < 64 ? 64 : g;
    const int upw = wave_k_of(K, g) / unit_k;
    const int nu = K / unit_k;
    const int max_units = 8 * upw;
    int ns = (nu + max_units - 1) / max_units;
    int ups = (nu + ns - 1) / ns;
    ups = (ups + upw - 1) / upw * upw;
    *nsplit = (nu + ups - 1) / ups;
    *units_per_split = ups;
}

}  // namespace

tq_status tqi_setup_skinny()
{
    bool ok = true;
#define TQ_ATTR(ST, GS, CW, WK, NW)                                                                                    \
    ok = ok && hipFuncSetAttribute((const void*)moe_skinny_kernel<ST, GS, CW, WK, NW>,                                    \
                                   hipFuncAttributeMaxDynamicSharedMemorySize, SK_LDS) == hipSuccess
#define TQ_ONE(ST, GS, CW) TQ_ATTR(ST, GS, CW, 512, 8); TQ_ATTR(ST, GS, CW, 256, 8); TQ_ATTR(ST, GS, CW, 256, 4); TQ_ATTR(ST, GS, CW, 256, 2)
    TQ_ONE(0, 2, 4); TQ_ONE(0, 4, 4); TQ_ONE(0, 8, 4); TQ_ONE(0, 16, 4);
    TQ_ONE(1, 2, 4); TQ_ONE(1, 4, 4); TQ_ONE(1, 8, 4); TQ_ONE(1, 16, 4);
    TQ_ONE(0, 4, 3); TQ_ONE(0, 8, 3); TQ_ONE(1, 4, 3); TQ_ONE(1, 8, 3);
    TQ_ONE(0, 4, 2); TQ_ONE(0, 8, 2); TQ_ONE(1, 4, 2); TQ_ONE(1, 8, 2);
#undef TQ_ONE
#undef TQ_ATTR
    return ok ? TQ_OK : TQ_ERR_HIP;
}

// Whether the decode path can run this layer (LDS budget, one workgroup must span the whole hidden size).
bool tqi_skinny_supported(const TqLayout& L)
{
    if (L.r16 > 64) return false;
    if (L.cw != 4 && L.g != 64 && L.g != 128) return false;
    int ns, ups;
    plan_split(L.H, L.g, &ns, &ups);
    if (ns != 1) return false;
    const int unit_k = L.g < 64 ? 64 : L.g;
    auto smem = [&](int units) {
        const int range_k = units * unit_k;
        return (size_t)16 * (range_k * 2 + 16) + sk_red_bytes(8) + (size_t)(range_k / L.g) * 64 + 16;
    };
    if (smem(ups) > SK_LDS) return false;
    plan_split(L.F, L.g, &ns, &ups);
    if (ns > TQ_MAX_SPLIT || smem(ups) > SK_LDS) return false;
    return true;
}

tq_status tqi_forward_skinny(const TqLayout& L, const TqWorkspace& W, const uint8_t* blob, const uint16_t* x,
                             int32_t T, uint8_t* ws, hipStream_t stream, int* nsplit_out)
{
    MGeom G;
    G.ne = L.E + L.S; G.H = L.H; G.F = L.F; G.g = L.g; G.r = L.r; G.r16 = L.r16; G.k = L.k; G.S = L.S;
    G.a_tot = W.a_tot; G.expert_stride = L.expert_stride; G.fm = L.fm;
    G.unpack_mask = L.cw == 4 ? 0x000F000Fu : L.cw == 3 ? 0x00070007u : 0x00030003u;
    G.unpack_magic = 0x43004300u;
    G.zc_ws = nullptr; G.zc_stride = 0; G.zc_d_off = 0;
    const int32_t* ctrl = reinterpret_cast<const int32_t*>(ws + W.ctrl);
    const int32_t* row_token = reinterpret_cast<const int32_t*>(ws + W.row_token);
    const int32_t* tile_e = reinterpret_cast<const int32_t*>(ws + W.tile_e) + 2 * (size_t)W.rt_max;      // 16-row tiling
    const int32_t* tile_row0 = reinterpret_cast<const int32_t*>(ws + W.tile_row0) + 2 * (size_t)W.rt_max;
    const int32_t* tile_rows = tile_row0 + (size_t)TQ_N_TILINGS * W.rt_max;      // row counts of the same tiling
    uint16_t* h = reinterpret_cast<uint16_t*>(ws + W.h);
    float* yd = reinterpret_cast<float*>(ws + W.yd);
    float* tpart = reinterpret_cast<float*>(ws + W.tpart);
    const int gs = L.g / 16;
    const int rt16 = W.a_tot / 16 + L.E + L.S;

    int ns, ups;
    plan_split(L.H, L.g, &ns, &ups);
    const int unit_k = L.g < 64 ? 64 : L.g;
    // parts of the intermediate in a split's range
    auto parts = [&](const TqSection& sec) { return (std::min(ups * unit_k, sec.K) + SK_PART_K - 1) / SK_PART_K; };
    auto pre = [&](auto kernel, const TqSection& sec, const uint16_t* xin) {
        hipLaunchKernelGGL(kernel, dim3(rt16, ns * parts(sec), sec.na_tiles), dim3(64 * TQ_PRE_PART_SLICES), 0, stream, G, sec, blob, xin,
                           row_token, tile_e, tile_row0, tile_rows, ctrl, tpart, ups * unit_k, parts(sec));
    };
    // decode batches proper: that of gate/up was computed per assignment in the permutation's launch
    const bool by_assign = tqi_pre_by_assign(L, W);
    const int32_t* row_src = by_assign ? reinterpret_cast<const int32_t*>(ws + W.row_src) : nullptr;
    if (L.r > 0 && !by_assign) {
        if (L.fm.fp8) pre(skinny_pre_kernel<0, true>, L.gu, x);
        else pre(skinny_pre_kernel<0, false>, L.gu, x);
        TQ_CHECK_LAUNCH();
    }
    tqi_record_stage(2, stream);
    int32_t* pair_cnt = reinterpret_cast<int32_t*>(ws + W.sk_cnt);
    if (W.sk_cnt_n < 2 * W.rt_max * TQ_MAX_SPLIT) return TQ_ERR_UNSUPPORTED;
    tq_status rc = launch_skinny_gs<0>(gs, L.cw, G, L.gu, blob, x, row_token, tile_e, tile_row0, tile_rows, ctrl, tpart, parts(L.gu), h, pair_cnt, rt16, 1,
                                       ups, stream, row_src, wave_k_of(L.H, L.g), waves_of(L.H, L.g));
    if (rc != TQ_OK) return rc;
    tqi_record_stage(3, stream);
    plan_split(L.F, L.g, &ns, &ups);
    if (L.r > 0) {
        if (L.fm.fp8) pre(skinny_pre_kernel<1, true>, L.d, h);
        else pre(skinny_pre_kernel<1, false>, L.d, h);
        TQ_CHECK_LAUNCH();
    }
    tqi_record_stage(4, stream);
    rc = launch_skinny_gs<1>(gs, L.cw, G, L.d, blob, h, row_token, tile_e, tile_row0, tile_rows, ctrl, tpart, parts(L.d), yd,
                             pair_cnt + (size_t)W.rt_max * TQ_MAX_SPLIT, rt16, ns, ups, stream, nullptr, wave_k_of(L.F, L.g), waves_of(L.F, L.g));
    if (rc != TQ_OK) return rc;
    *nsplit_out = ns;
    return TQ_OK;
}
