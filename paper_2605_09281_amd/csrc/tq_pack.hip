// tq_pack_weights / tq_unpack_weights: canonical expert weights <-> the packed blob whose layout
// include/tileq.h specifies.  Pure index arithmetic; every element is moved bit for bit.
#include "tq_prep.h"

namespace {

using tqprep::PackGeom;
using tqprep::make_geom;
using tqprep::zc_part;
using tqdev::u32x4;

// Codes: a workgroup moves a span of up to eight 64-wide chunks of one column pair (64 canonical rows) between the
// canonical bytes and the packed words, through LDS.  Bound by memory: canonical rows are read (written) in runs of
// 512 bytes and the packed side in runs of 1 KB (CW x 256 bytes for dense codes), 128 bytes per thread in flight.  One
// thread per packed word, which reads 8 bytes of a row of its own, measured 900 us on 8 experts of 4096 x 14336 (1.41 GB of
// bytes to 0.70 GB of words: 2.3 TB/s); this form 339 us
// (6.2 TB/s).  Rows shorter than eight chunks leave some of the loading threads idle: whole call on 128 experts of
// 1024 x 512 207 us before, 88 now, on 64 of 512 x 256 (dense 2-bit codes) 28 / 18, on 8 of 256 x 512 19 / 12.
// Row stride in LDS: 528 bytes is the 16-byte alignment that the b128 accesses need, and leaves two rows of 16 apart (of the 32
// that a wave reads 8 bytes of at a time) on the same banks.
constexpr int PK_CHUNKS = 8, PK_ROWB = 64 * PK_CHUNKS + 16;

// the 32 codes of (pair, chunk, tile, lane) <-> CW words; v[w] = codes kk = 16 w + 8 hf + (0..7) as bytes
template <int CW>
__device__ inline void codes_to_words(const uint64_t (&v)[4], uint32_t (&word)[CW])
{
#pragma unroll
    for (int d = 0; d < CW; ++d) word[d] = 0;
#pragma unroll
    for (int ws = 0; ws < 4; ++ws) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t lo = (uint32_t)(v[ws] >> (16 * j)) & 0xFF, hi = (uint32_t)(v[ws] >> (16 * j + 8)) & 0xFF;
            const int P = 4 * ws + j;
            if constexpr (CW == 4) {
                word[ws] |= (lo & 15u) << (4 * tq_nibble_pos(2 * j)) | (hi & 15u) << (4 * tq_nibble_pos(2 * j + 1));
            } else if constexpr (CW == 2) {
                word[P / 8] |= ((lo & 3u) | ((hi & 3u) << 16)) << (2 * (P % 8));
            } else if (P < 15) {
                word[P / 5] |= ((lo & 7u) | ((hi & 7u) << 16)) << (3 * (P % 5));
            } else {
#pragma unroll
                for (int b = 0; b < 3; ++b) word[b % CW] |= (((lo >> b) & 1u) << 15) | (((hi >> b) & 1u) << 31);
            }
        }
    }
}

template <int CW>
__device__ inline void words_to_codes(const uint32_t (&word)[CW], uint64_t (&v)[4])
{
#pragma unroll
    for (int ws = 0; ws < 4; ++ws) {
        v[ws] = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int P = 4 * ws + j;
            uint32_t lo, hi;
            if constexpr (CW == 4) {
                lo = (word[ws] >> (4 * tq_nibble_pos(2 * j))) & 15u;
                hi = (word[ws] >> (4 * tq_nibble_pos(2 * j + 1))) & 15u;
            } else if constexpr (CW == 2) {
                const uint32_t t = word[P / 8] >> (2 * (P % 8));
                lo = t & 3u; hi = (t >> 16) & 3u;
            } else if (P < 15) {
                const uint32_t t = word[P / 5] >> (3 * (P % 5));
                lo = t & 7u; hi = (t >> 16) & 7u;
            } else {
                lo = hi = 0;
#pragma unroll
                for (int b = 0; b < 3; ++b) {
                    lo |= ((word[b % CW] >> 15) & 1u) << b;
                    hi |= ((word[b % CW] >> 31) & 1u) << b;
                }
            }
            v[ws] |= (uint64_t)lo << (16 * j) | (uint64_t)hi << (16 * j + 8);
        }
    }
}

template <bool PACK, int CW>
__global__ void __launch_bounds__(256) codes_kernel(PackGeom G, uint8_t* __restrict__ blob, uint8_t* __restrict__ codes,
                                                    int32_t* __restrict__ err_flag)
{
    __shared__ __attribute__((aligned(16))) uint8_t lds[64 * PK_ROWB];
    const int spans_gu = (G.gu.chunks + PK_CHUNKS - 1) / PK_CHUNKS, spans_d = (G.d.chunks + PK_CHUNKS - 1) / PK_CHUNKS;
    const uint32_t n_gu = (uint32_t)G.gu.pairs * spans_gu, per_exp = n_gu + (uint32_t)G.d.pairs * spans_d;
    const int e = blockIdx.x / per_exp;
    uint32_t q = blockIdx.x % per_exp;
    const bool is_d = q >= n_gu;
    if (is_d) q -= n_gu;
    const TqSection& sec = is_d ? G.d : G.gu;
    const int spans = is_d ? spans_d : spans_gu;
    const int pair = q / spans, c0 = (q % spans) * PK_CHUNKS, nc = min(PK_CHUNKS, sec.chunks - c0);
    const int tid = threadIdx.x;
    const size_t HF = (size_t)G.H * G.F;
    // canonical row of LDS row `row` (tile row / 32, column row % 32 of the pair), at the span's first byte
    auto canon = [&](int row) {
        const int tile = row >> 5, p = is_d ? 2 : tile, n = is_d ? 64 * pair + row : 32 * pair + (row & 31);
        return codes + ((size_t)e * 3 + p) * HF + (size_t)n * sec.K + 64 * c0;
    };
    uint32_t* const words = reinterpret_cast<uint32_t*>(blob + TQ_HEADER_BYTES + (size_t)e * G.expert_stride + sec.codes) +
                            ((size_t)pair * sec.chunks + c0) * (2 * 64 * CW);
    constexpr int SEGS = 4 * PK_CHUNKS, NP = 64 * SEGS / 256;      // 16-byte segments per row; passes
    const int seg = tid % SEGS, row0 = tid / SEGS;
    const bool in = seg < 4 * nc;
    if (PACK) {
        u32x4 v[NP];
#pragma unroll
        for (int i = 0; i < NP; ++i)
            v[i] = in ? __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(canon(row0 + i * (256 / SEGS))) + seg) : u32x4{0u, 0u, 0u, 0u};
        uint32_t any = 0;
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            any |= v[i][0] | v[i][1] | v[i][2] | v[i][3];
            *reinterpret_cast<u32x4*>(lds + (row0 + i * (256 / SEGS)) * PK_ROWB + seg * 16) = v[i];
        }
        // qmax is 2^bits - 1: a code beyond it has a bit above
        if ((any & ((0xFFu & ~(uint32_t)G.qmax) * 0x01010101u)) && err_flag) atomicOr(err_flag, TQ_FLAG_BIT_RANGE);
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < PK_CHUNKS * 128 / 256; ++i) {
        const int job = i * 256 + tid, lane = job & 63, tile = (job >> 6) & 1, c = job >> 7;
        uint8_t* src = lds + (32 * tile + (lane & 31)) * PK_ROWB + 64 * c + 8 * (lane >> 5);
        if (c >= nc) break;
        uint64_t v[4];
        uint32_t word[CW];
        uint32_t* dst = words + (size_t)(c * 2 + tile) * (64 * CW);
        if (PACK) {
#pragma unroll
            for (int w = 0; w < 4; ++w) v[w] = *reinterpret_cast<const uint64_t*>(src + 16 * w);
            codes_to_words<CW>(v, word);
            if constexpr (CW == 4) {
                reinterpret_cast<u32x4*>(dst)[lane] = u32x4{word[0], word[1], word[2], word[3]};
            } else {
#pragma unroll
                for (int d = 0; d < CW; ++d) dst[64 * d + lane] = word[d];
            }
        } else {
            if constexpr (CW == 4) {
                const u32x4 t = reinterpret_cast<const u32x4*>(dst)[lane];
#pragma unroll
                for (int d = 0; d < 4; ++d) word[d] = t[d];
            } else {
#pragma unroll
                for (int d = 0; d < CW; ++d) word[d] = dst[64 * d + lane];
            }
            words_to_codes<CW>(word, v);
#pragma unroll
            for (int w = 0; w < 4; ++w) *reinterpret_cast<uint64_t*>(src + 16 * w) = v[w];
        }
    }
    if (!PACK) {
        __syncthreads();
        if (in) {
#pragma unroll
            for (int i = 0; i < NP; ++i)
                reinterpret_cast<u32x4*>(canon(row0 + i * (256 / SEGS)))[seg] =
                    *reinterpret_cast<const u32x4*>(lds + (row0 + i * (256 / SEGS)) * PK_ROWB + seg * 16);
        }
    }
}

// Scales and zero-points: a workgroup moves 64 groups of one column pair between the canonical rows and the sz words, and
// on packing derives the pair's zc fragments from the same values.  Bound by memory: canonical rows are read in runs of
// 128 bytes (one thread per word, strided by the number of groups, took 72 us for sz and another 90 us for zc on 8 experts of
// 4096 x 14336, groups of 128; this form 35 us for both).  Rows of fewer groups repeat the last one on the lanes past it; the whole
// call's times on such layers stand at PK_CHUNKS.
constexpr int SZ_GROUPS = 64;

template <bool PACK>
__global__ void __launch_bounds__(256) sz_kernel(PackGeom G, uint8_t* __restrict__ blob, uint16_t* __restrict__ scale,
                                                 uint16_t* __restrict__ zero, TqBlobHeader hdr)
{
    __shared__ uint32_t lds[64][SZ_GROUPS + 1];      // the odd stride spreads a column over the banks
    const int spans_gu = (G.gu.groups + SZ_GROUPS - 1) / SZ_GROUPS, spans_d = (G.d.groups + SZ_GROUPS - 1) / SZ_GROUPS;
    const uint32_t n_gu = (uint32_t)G.gu.pairs * spans_gu, per_exp = n_gu + (uint32_t)G.d.pairs * spans_d;
    const int e = blockIdx.x / per_exp;
    uint32_t q = blockIdx.x % per_exp;
    const bool is_d = q >= n_gu;
    if (is_d) q -= n_gu;
    const TqSection& sec = is_d ? G.d : G.gu;
    const int spans = is_d ? spans_d : spans_gu;
    const int pair = q / spans, g0 = (q % spans) * SZ_GROUPS, ng = min(SZ_GROUPS, sec.groups - g0);
    const int tid = threadIdx.x;
    if (PACK && blockIdx.x == 0 && tid == 0) *reinterpret_cast<TqBlobHeader*>(blob) = hdr;      // (saves a launch)
    const size_t HFg = (size_t)G.H * G.F / G.g;
    auto canon = [&](int row) {      // index of group g0 of LDS row `row` (tile row / 32, column row % 32)
        const int tile = row >> 5, p = is_d ? 2 : tile, n = is_d ? 64 * pair + row : 32 * pair + (row & 31);
        return ((size_t)e * 3 + p) * HFg + (size_t)n * sec.groups + g0;
    };
    uint32_t* const words = reinterpret_cast<uint32_t*>(blob + TQ_HEADER_BYTES + (size_t)e * G.expert_stride + sec.sz) +
                            ((size_t)pair * sec.groups + g0) * 64;
    const int gl = tid % SZ_GROUPS, row0 = tid / SZ_GROUPS;
    constexpr int NP = 64 * SZ_GROUPS / 256;
    if (PACK) {
        uint16_t sv[NP], zv[NP];
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            const size_t ci = canon(row0 + i * (256 / SZ_GROUPS)) + min(gl, ng - 1);
            sv[i] = scale[ci];
            zv[i] = zero[ci];
        }
#pragma unroll
        for (int i = 0; i < NP; ++i) lds[row0 + i * (256 / SZ_GROUPS)][gl] = (uint32_t)sv[i] | ((uint32_t)zv[i] << 16);
        __syncthreads();
    }
    for (int w = tid; w < ng * 64; w += 256) {      // word (group, tile, column)
        if (PACK) words[w] = lds[w & 63][w >> 6];
        else lds[w & 63][w >> 6] = words[w];
    }
    if (!PACK) {
        __syncthreads();
        if (gl < ng) {
#pragma unroll
            for (int i = 0; i < NP; ++i) {
                const size_t ci = canon(row0 + i * (256 / SZ_GROUPS)) + gl;
                const uint32_t v = lds[row0 + i * (256 / SZ_GROUPS)][gl];
                scale[ci] = (uint16_t)(v & 0xFFFF);
                zero[ci] = (uint16_t)(v >> 16);
            }
        }
    } else if (sec.zsteps > 0) {
        // fragments of this span's 16-group blocks: (block, hi | lo, tile, lane), 8 values each, 0 past the last group
        u32x4* dst = reinterpret_cast<u32x4*>(blob + TQ_HEADER_BYTES + (size_t)e * G.expert_stride + sec.zc) +
                     ((size_t)pair * sec.zsteps + 2 * (g0 / 16)) * 128;
        const int nf = 2 * ((ng + 15) / 16) * 128;
        for (int w = tid; w < nf; w += 256) {
            const int lane = w & 63, tile = (w >> 6) & 1, f = w >> 7, gb = 16 * (f >> 1) + 8 * (lane >> 5);
            uint32_t v[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = gb + i < ng ? zc_part(lds[32 * tile + (lane & 31)][min(gb + i, SZ_GROUPS - 1)], f & 1) : 0u;
            dst[w] = u32x4{v[0] | (v[1] << 16), v[2] | (v[3] << 16), v[4] | (v[5] << 16), v[6] | (v[7] << 16)};
        }
    }
}

// Factor fragments, one thread per 8-element fragment (B's in front of A's: one launch for both).
// B: padding rows (rho >= r) are written as zero and skipped on unpack.
// ET: uint16_t (fp16 bit patterns) or uint8_t (fp8 E4M3 codes): the layout is the same with 2- or 1-byte elements.
template <bool PACK, typename ET>
__device__ inline void bfrag_one(const PackGeom& G, uint8_t* __restrict__ blob, ET* __restrict__ B, size_t idx)
{
    const int steps = G.r16 / 16;
    const size_t n_gu = (size_t)G.gu.pairs * steps * 128;
    const size_t n_d = (size_t)G.d.pairs * steps * 128;
    const size_t per_exp = n_gu + n_d;
    int e = (int)(idx / per_exp);
    size_t w = idx % per_exp;
    const bool is_d = w >= n_gu;
    const TqSection& sec = is_d ? G.d : G.gu;
    if (is_d) w -= n_gu;
    int lane = (int)(w & 63);
    int tile = (int)((w >> 6) & 1);
    size_t ps = w >> 7;
    int step = (int)(ps % steps);
    int pair = (int)(ps / steps);
    int col = lane & 31, hf = lane >> 5;
    int p, n, N;
    if (!is_d) { p = tile; n = 32 * pair + col; N = G.F; }
    else       { p = 2;    n = 64 * pair + 32 * tile + col; N = G.H; }
    const size_t b_per_exp = (2 * (size_t)G.F + G.H) * G.r;
    const size_t b_off = (p == 0) ? 0 : (p == 1) ? (size_t)G.F * G.r : 2 * (size_t)G.F * G.r;
    ET* src = B + (size_t)e * b_per_exp + b_off;
    ET* dst = reinterpret_cast<ET*>(blob + TQ_HEADER_BYTES + (size_t)e * G.expert_stride + sec.bfrag) + w * 8;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        int rho = 16 * step + 8 * hf + i;
        if (PACK) dst[i] = (rho < G.r) ? src[(size_t)rho * N + n] : (ET)0;
        else if (rho < G.r) src[(size_t)rho * N + n] = dst[i];
    }
}

// A: padding columns (c >= NA or rho >= r) likewise.
template <bool PACK, typename ET>
__device__ inline void afrag_one(const PackGeom& G, uint8_t* __restrict__ blob, ET* __restrict__ A, size_t idx)
{
    const size_t n_gu = (size_t)G.gu.na_tiles * (G.gu.K / 16) * 64;
    const size_t n_d = (size_t)G.d.na_tiles * (G.d.K / 16) * 64;
    const size_t per_exp = n_gu + n_d;
    int e = (int)(idx / per_exp);
    size_t w = idx % per_exp;
    const bool is_d = w >= n_gu;
    const TqSection& sec = is_d ? G.d : G.gu;
    if (is_d) w -= n_gu;
    int lane = (int)(w & 63);
    size_t ts = w >> 6;
    int ksteps = sec.K / 16;
    int step = (int)(ts % ksteps);
    int ta = (int)(ts / ksteps);
    int c = 32 * ta + (lane & 31), hf = lane >> 5;
    int na = is_d ? G.r16 : 2 * G.r16;
    int p = is_d ? 2 : (c / G.r16);
    int rho = c % G.r16;
    const bool live = (c < na) && (rho < G.r);
    const size_t a_per_exp = (2 * (size_t)G.H + G.F) * G.r;
    const size_t a_off = (p == 0) ? 0 : (p == 1) ? (size_t)G.H * G.r : 2 * (size_t)G.H * G.r;
    ET* src = A + (size_t)e * a_per_exp + a_off;
    ET* dst = reinterpret_cast<ET*>(blob + TQ_HEADER_BYTES + (size_t)e * G.expert_stride + sec.afrag) + w * 8;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        int kk = 16 * step + 8 * hf + i;
        if (PACK) dst[i] = live ? src[(size_t)kk * G.r + rho] : (ET)0;
        else if (live) src[(size_t)kk * G.r + rho] = dst[i];
    }
}

template <bool PACK, typename ET>
__global__ void __launch_bounds__(256) factors_kernel(PackGeom G, uint8_t* __restrict__ blob, ET* __restrict__ A, ET* __restrict__ B,
                                                      size_t n_b, size_t n_a)
{
    const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx < n_b) bfrag_one<PACK>(G, blob, B, idx);
    else if (idx < n_b + n_a) afrag_one<PACK>(G, blob, A, idx - n_b);
}

// Sigma of fp8 factors: fp16 [n_exp][3][r] <-> the fp32 `sig` parts of the records (GU: gate then up, r16 each; D),
// each padded with zeros to 256 bytes.  With n_tables == 1 and shared factors the one table [3][r] goes behind the pools.
template <bool PACK>
__global__ void sig_kernel(PackGeom G, TqFactorMap fm, uint8_t* __restrict__ blob, uint16_t* __restrict__ sigma, int n_tables)
{
    const int n_gu = (int)(tq_align256((size_t)2 * G.r16 * 4) / 4), n_d = (int)(tq_align256((size_t)G.r16 * 4) / 4);
    const int per = n_gu + n_d;
    const int idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= per * n_tables) return;
    const int e = idx / per;
    int c = idx % per;
    const bool is_d = c >= n_gu;
    if (is_d) c -= n_gu;
    const TqSection& sec = is_d ? G.d : G.gu;
    float* dst = (fm.shared ? reinterpret_cast<float*>(blob + fm.sig_off[is_d])
                            : reinterpret_cast<float*>(blob + TQ_HEADER_BYTES + (size_t)e * G.expert_stride + sec.sig)) + c;
    const int p = is_d ? 2 : c / G.r16, rho = c % G.r16;
    const bool live = c < (is_d ? G.r16 : 2 * G.r16) && rho < G.r;
    uint16_t* src = sigma + ((size_t)e * 3 + p) * G.r + rho;
    if (PACK) *dst = live ? __half2float(__ushort_as_half(*src)) : 0.f;
    else if (live) *src = __half_as_ushort(__float2half(*dst));      // exact: the value came from an fp16
}

// Shared 2D-tiled factors.  Left factors: one thread per 8-element fragment of block (section, m); the block has the
// afrag layout, its columns being [gate factor | up factor] (r16 each) in section GU and the down factor in D.
template <typename ET>
__global__ void pool_afrag_kernel(PackGeom G, TqFactorMap fm, uint8_t* __restrict__ blob,
                                  const ET* __restrict__ us_g, const ET* __restrict__ us_u,
                                  const ET* __restrict__ us_d)
{
    const size_t n_gu = (size_t)G.gu.na_tiles * (G.gu.K / 16) * 64;     // fragments per block
    const size_t n_d = (size_t)G.d.na_tiles * (G.d.K / 16) * 64;
    const size_t per_m = n_gu + n_d;
    size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= per_m * fm.M) return;
    const int m = (int)(idx / per_m);
    size_t w = idx % per_m;
    const bool is_d = w >= n_gu;
    const TqSection& sec = is_d ? G.d : G.gu;
    if (is_d) w -= n_gu;
    const int lane = (int)(w & 63);
    const size_t ts = w >> 6;
    const int ksteps = sec.K / 16;
    const int step = (int)(ts % ksteps), ta = (int)(ts / ksteps);
    const int c = 32 * ta + (lane & 31), hf = lane >> 5;
    const int na = is_d ? G.r16 : 2 * G.r16;
    const int p = is_d ? 2 : (c / G.r16);
    const int rho = c % G.r16;
    const bool live = (c < na) && (rho < G.r);
    const ET* src = (p == 0 ? us_g : p == 1 ? us_u : us_d) + (size_t)m * sec.K * G.r;      // [K][r] of tile row m
    ET* dst = reinterpret_cast<ET*>(blob + fm.apool[is_d] + (size_t)m * fm.astride[is_d]) + w * 8;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int kk = 16 * step + 8 * hf + i;
        dst[i] = live ? src[(size_t)kk * G.r + rho] : (ET)0;
    }
}

// Right factors: one thread per 8-element fragment of block (section, n), in the bfrag layout (tile 0 / 1 of a pair:
// gate / up factor in section GU, the two 32-column halves of the down factor's 64 columns in D).
template <typename ET>
__global__ void pool_bfrag_kernel(PackGeom G, TqFactorMap fm, uint8_t* __restrict__ blob,
                                  const ET* __restrict__ v_g, const ET* __restrict__ v_u,
                                  const ET* __restrict__ v_d)
{
    const int steps = G.r16 / 16;
    const size_t n_gu = (size_t)G.gu.pairs * steps * 128;
    const size_t n_d = (size_t)G.d.pairs * steps * 128;
    const size_t per_n = n_gu + n_d;
    size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= per_n * fm.N) return;
    const int nt = (int)(idx / per_n);
    size_t w = idx % per_n;
    const bool is_d = w >= n_gu;
    if (is_d) w -= n_gu;
    const int lane = (int)(w & 63), tile = (int)((w >> 6) & 1);
    const size_t ps = w >> 7;
    const int step = (int)(ps % steps), pair = (int)(ps / steps);
    const int col = lane & 31, hf = lane >> 5;
    int p, n, N;
    if (!is_d) { p = tile; n = 32 * pair + col; N = G.F; }
    else       { p = 2;    n = 64 * pair + 32 * tile + col; N = G.H; }
    const ET* src = (p == 0 ? v_g : p == 1 ? v_u : v_d) + (size_t)nt * G.r * N;              // [r][N] of tile column nt
    ET* dst = reinterpret_cast<ET*>(blob + fm.bpool[is_d] + (size_t)nt * fm.bstride[is_d]) + w * 8;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int rho = 16 * step + 8 * hf + i;
        dst[i] = (rho < G.r) ? src[(size_t)rho * N + n] : (ET)0;
    }
}

__global__ void phi_kernel(TqFactorMap fm, int n_exp, int n_padded, uint8_t* __restrict__ blob, const int32_t* __restrict__ phi,
                           int32_t* __restrict__ err_flag)
{
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n_padded) return;
    int m = 0, n = 0;                    // entries of the padding behind the table are written as zeros
    if (e < n_exp) {
        m = phi[2 * e]; n = phi[2 * e + 1];
        if (m < 0 || m >= fm.M || n < 0 || n >= fm.N) {
            if (err_flag) atomicOr(err_flag, TQ_FLAG_BIT_RANGE);
            m = min(max(m, 0), fm.M - 1);
            n = min(max(n, 0), fm.N - 1);
        }
    }
    int32_t* dst = reinterpret_cast<int32_t*>(blob + fm.phi_off);
    dst[2 * e] = m;
    dst[2 * e + 1] = n;
}

inline unsigned blocks_for(size_t n) { return (unsigned)((n + 255) / 256); }

template <bool PACK>
tq_status run(const TqLayout& L, uint8_t* blob, uint8_t* codes, uint16_t* scale, uint16_t* zero,
              uint16_t* A, uint16_t* B, uint16_t* sigma, int32_t* err_flag, hipStream_t st, const TqBlobHeader& hdr = {})
{
    PackGeom G = make_geom(L);
    const size_t ne = G.n_exp;
    auto spans = [](int n, int per) { return (size_t)((n + per - 1) / per); };
    const size_t n_codes = (L.gu.pairs * spans(L.gu.chunks, PK_CHUNKS) + L.d.pairs * spans(L.d.chunks, PK_CHUNKS)) * ne;
    const size_t n_sz = (L.gu.pairs * spans(L.gu.groups, SZ_GROUPS) + L.d.pairs * spans(L.d.groups, SZ_GROUPS)) * ne;
    if (n_codes > 0x7FFFFFFFull || n_sz > 0x7FFFFFFFull) return TQ_ERR_UNSUPPORTED;
    if (L.cw == 4)
        hipLaunchKernelGGL((codes_kernel<PACK, 4>), dim3((unsigned)n_codes), dim3(256), 0, st, G, blob, codes, err_flag);
    else if (L.cw == 3)
        hipLaunchKernelGGL((codes_kernel<PACK, 3>), dim3((unsigned)n_codes), dim3(256), 0, st, G, blob, codes, err_flag);
    else
        hipLaunchKernelGGL((codes_kernel<PACK, 2>), dim3((unsigned)n_codes), dim3(256), 0, st, G, blob, codes, err_flag);
    TQ_CHECK_LAUNCH();
    hipLaunchKernelGGL(sz_kernel<PACK>, dim3((unsigned)n_sz), dim3(256), 0, st, G, blob, scale, zero, hdr);
    TQ_CHECK_LAUNCH();
    if (L.r > 0 && !L.fm.shared) {
        size_t n_b = ((size_t)L.gu.pairs + L.d.pairs) * (L.r16 / 16) * 128 * ne;
        size_t n_a = ((size_t)L.gu.na_tiles * (L.gu.K / 16) + (size_t)L.d.na_tiles * (L.d.K / 16)) * 64 * ne;
        if (L.fm.fp8) {
            hipLaunchKernelGGL((factors_kernel<PACK, uint8_t>), dim3(blocks_for(n_b + n_a)), dim3(256), 0, st, G, blob, (uint8_t*)A,
                               (uint8_t*)B, n_b, n_a);
            TQ_CHECK_LAUNCH();
            hipLaunchKernelGGL(sig_kernel<PACK>, dim3(blocks_for((tq_align256((size_t)8 * L.r16) + tq_align256((size_t)4 * L.r16)) / 4 * ne)),
                               dim3(256), 0, st, G, L.fm, blob, sigma, (int)ne);
            TQ_CHECK_LAUNCH();
        } else {
            hipLaunchKernelGGL((factors_kernel<PACK, uint16_t>), dim3(blocks_for(n_b + n_a)), dim3(256), 0, st, G, blob, A, B, n_b, n_a);
            TQ_CHECK_LAUNCH();
        }
    }
    return TQ_OK;
}

inline bool misaligned(const void* p, size_t a) { return ((uintptr_t)p & (a - 1)) != 0; }

}  // namespace

tq_status tqi_make_prep(const TqLayout& L, const TqWorkspace& W, const uint8_t* blob, uint8_t* ws, TqPrep* P)
{
    const bool factors = L.fm.fp8 != 0, zc = L.cw != 4;
    P->n_waves = 0;
    if ((factors && W.fac_bytes == 0) || (zc && W.zc_stride == 0)) return TQ_ERR_UNSUPPORTED;
    if (!factors && !zc) return TQ_OK;
    P->G = make_geom(L);
    P->src = L.fm; P->dstm = W.fac_fm;
    P->blob = blob; P->fbase = ws + W.fac_ws; P->zc_ws = ws + W.zc_ws;
    P->zc_stride = W.zc_stride; P->zc_d_off = W.zc_d_off;
    size_t n = 0;
    auto part = [&](int i, size_t threads) { n += (threads + 63) / 64; P->end[i] = (unsigned)n; };
    const size_t ne = L.E + L.S;
    part(0, factors ? ne : 0);
    part(1, factors ? (((size_t)L.gu.na_tiles * (L.gu.K / 16) + (size_t)L.d.na_tiles * (L.d.K / 16)) * 64) * W.fac_fm.M : 0);
    part(2, factors ? (((size_t)L.gu.pairs + L.d.pairs) * (L.r16 / 16) * 128) * W.fac_fm.N : 0);
    part(3, zc ? ((size_t)L.gu.pairs * (L.gu.zfrag / 2) + (size_t)L.d.pairs * (L.d.zfrag / 2)) * 128 * ne : 0);
    if (n > 0x3FFFFFFF) return TQ_ERR_UNSUPPORTED;
    P->n_waves = (unsigned)n;
    return TQ_OK;
}

extern "C" size_t tq_packed_size(const tq_layer_desc* desc)
{
    TqLayout L;
    if (!tq_make_layout(desc, &L)) return 0;
    return L.total_bytes;
}

namespace {
tq_status pack_impl(const tq_layer_desc* desc, const tq_weights_src* src, const tq_shared_factors* shared, void* packed,
                    size_t packed_bytes, int32_t* err_flag, void* stream);
}

extern "C" tq_status tq_pack_weights(const tq_layer_desc* desc, const tq_weights_src* src, void* packed,
                                     size_t packed_bytes, int32_t* err_flag, void* stream)
{
    if (desc && (desc->tiles_m || desc->tiles_n)) return TQ_ERR_SHAPE;      // shared factors: tq_pack_weights_shared
    return pack_impl(desc, src, nullptr, packed, packed_bytes, err_flag, stream);
}

extern "C" tq_status tq_pack_weights_shared(const tq_layer_desc* desc, const tq_weights_src* src,
                                            const tq_shared_factors* shared, void* packed, size_t packed_bytes,
                                            int32_t* err_flag, void* stream)
{
    if (!shared) return TQ_ERR_NULL;
    if (desc && !(desc->tiles_m > 0 && desc->tiles_n > 0)) return TQ_ERR_SHAPE;
    for (int p = 0; p < 3; ++p) {
        if (!shared->us[p] || !shared->v[p]) return TQ_ERR_NULL;
        if ((((uintptr_t)shared->us[p]) | ((uintptr_t)shared->v[p])) & 15) return TQ_ERR_ALIGN;
    }
    if (!shared->phi) return TQ_ERR_NULL;
    if ((uintptr_t)shared->phi & 3) return TQ_ERR_ALIGN;
    return pack_impl(desc, src, shared, packed, packed_bytes, err_flag, stream);
}

namespace {
tq_status pack_impl(const tq_layer_desc* desc, const tq_weights_src* src, const tq_shared_factors* shared, void* packed,
                    size_t packed_bytes, int32_t* err_flag, void* stream)
{
    if (!desc || !src || !packed || !src->codes || !src->scale || !src->zero) return TQ_ERR_NULL;
    TqLayout L;
    if (!tq_make_layout(desc, &L)) return TQ_ERR_SHAPE;
    if (L.r > 0 && !L.fm.shared && (!src->A || !src->B)) return TQ_ERR_NULL;
    if (L.fm.fp8 && !(L.fm.shared ? shared->sigma : src->sigma)) return TQ_ERR_NULL;
    if (L.fm.fp8 && misaligned(L.fm.shared ? shared->sigma : src->sigma, 2)) return TQ_ERR_ALIGN;
    if (packed_bytes < L.total_bytes) return TQ_ERR_WORKSPACE;
    if (misaligned(packed, 256) || misaligned(src->codes, 16) || misaligned(src->scale, 16) ||
        misaligned(src->zero, 16) || (L.r > 0 && !L.fm.shared && (misaligned(src->A, 16) || misaligned(src->B, 16))) ||
        misaligned(err_flag, 4))
        return TQ_ERR_ALIGN;
    hipStream_t st = (hipStream_t)stream;
    TqBlobHeader hdr = {};
    hdr.magic = TQ_BLOB_MAGIC; hdr.version = TQ_BLOB_VERSION;
    hdr.n_experts = L.E; hdr.n_shared = L.S; hdr.hidden = L.H; hdr.ffn = L.F; hdr.group = L.g;
    hdr.bits = L.bits; hdr.rank = L.r; hdr.r16 = L.r16; hdr.code_words = L.cw; hdr.factor_fp8 = L.fm.fp8;
    hdr.tiles_m = L.fm.M; hdr.tiles_n = L.fm.N;
    hdr.expert_stride = L.expert_stride; hdr.total_bytes = L.total_bytes;
    hdr.off[0] = L.gu.codes; hdr.off[1] = L.gu.sz; hdr.off[2] = L.gu.zc; hdr.off[3] = L.gu.bfrag; hdr.off[4] = L.gu.afrag;
    hdr.off[5] = L.d.codes; hdr.off[6] = L.d.sz; hdr.off[7] = L.d.zc; hdr.off[8] = L.d.bfrag; hdr.off[9] = L.d.afrag;
    tq_status rc = run<true>(L, (uint8_t*)packed, const_cast<uint8_t*>(src->codes), const_cast<uint16_t*>(src->scale),
                             const_cast<uint16_t*>(src->zero), const_cast<uint16_t*>(src->A),
                             const_cast<uint16_t*>(src->B), const_cast<uint16_t*>(src->sigma), err_flag, st, hdr);
    if (rc != TQ_OK || !L.fm.shared) return rc;
    const PackGeom G = make_geom(L);
    const size_t n_a = ((size_t)L.gu.na_tiles * (L.gu.K / 16) + (size_t)L.d.na_tiles * (L.d.K / 16)) * 64 * L.fm.M;
    const size_t n_b = ((size_t)L.gu.pairs + L.d.pairs) * (L.r16 / 16) * 128 * L.fm.N;
    if (L.fm.fp8) {
        hipLaunchKernelGGL(pool_afrag_kernel<uint8_t>, dim3(blocks_for(n_a)), dim3(256), 0, st, G, L.fm, (uint8_t*)packed,
                           (const uint8_t*)shared->us[0], (const uint8_t*)shared->us[1], (const uint8_t*)shared->us[2]);
        TQ_CHECK_LAUNCH();
        hipLaunchKernelGGL(pool_bfrag_kernel<uint8_t>, dim3(blocks_for(n_b)), dim3(256), 0, st, G, L.fm, (uint8_t*)packed,
                           (const uint8_t*)shared->v[0], (const uint8_t*)shared->v[1], (const uint8_t*)shared->v[2]);
        TQ_CHECK_LAUNCH();
        hipLaunchKernelGGL(sig_kernel<true>, dim3(blocks_for((tq_align256((size_t)8 * L.r16) + tq_align256((size_t)4 * L.r16)) / 4)),
                           dim3(256), 0, st, G, L.fm, (uint8_t*)packed, const_cast<uint16_t*>(shared->sigma), 1);
        TQ_CHECK_LAUNCH();
    } else {
        hipLaunchKernelGGL(pool_afrag_kernel<uint16_t>, dim3(blocks_for(n_a)), dim3(256), 0, st, G, L.fm, (uint8_t*)packed,
                           shared->us[0], shared->us[1], shared->us[2]);
        TQ_CHECK_LAUNCH();
        hipLaunchKernelGGL(pool_bfrag_kernel<uint16_t>, dim3(blocks_for(n_b)), dim3(256), 0, st, G, L.fm, (uint8_t*)packed,
                           shared->v[0], shared->v[1], shared->v[2]);
        TQ_CHECK_LAUNCH();
    }
    const int n_padded = (int)(tq_align256((size_t)(L.E + L.S) * 8) / 8);
    hipLaunchKernelGGL(phi_kernel, dim3(blocks_for((size_t)n_padded)), dim3(256), 0, st, L.fm, L.E + L.S, n_padded,
                       (uint8_t*)packed, shared->phi, err_flag);
    TQ_CHECK_LAUNCH();
    return TQ_OK;
}
}  // namespace

extern "C" tq_status tq_unpack_weights(const tq_layer_desc* desc, const void* packed, const tq_weights_dst* dst,
                                       void* stream)
{
    if (!desc || !dst || !packed || !dst->codes || !dst->scale || !dst->zero) return TQ_ERR_NULL;
    TqLayout L;
    if (!tq_make_layout(desc, &L)) return TQ_ERR_SHAPE;
    if (L.r > 0 && !L.fm.shared && (!dst->A || !dst->B)) return TQ_ERR_NULL;      // shared factors: codes, scale, zero only
    if (L.fm.fp8 && !L.fm.shared && (!dst->sigma || misaligned(dst->sigma, 2))) return TQ_ERR_NULL;
    if (misaligned(packed, 256) || misaligned(dst->codes, 16) || misaligned(dst->scale, 16) ||
        misaligned(dst->zero, 16) || (L.r > 0 && !L.fm.shared && (misaligned(dst->A, 16) || misaligned(dst->B, 16))))
        return TQ_ERR_ALIGN;
    return run<false>(L, const_cast<uint8_t*>((const uint8_t*)packed), dst->codes, dst->scale, dst->zero, dst->A,
                      dst->B, dst->sigma, nullptr, (hipStream_t)stream);
}
