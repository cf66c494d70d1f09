// Offline helper: rank-r approximation of a dense fp32 matrix by r Gaussian-sketch rank-1 deflations (Section 3.1,
// "Plug-in", Eq. 13), the replacement for the SVD of the tiled matrix W_big of Eq. 11.  Per rank, with sketch vector s:
//   Q = (W W^T)^it W s,   U = Q / |Q|,   Sigma = |Q^T W| / |Q|,   V = Q^T W / |Q^T W|,   W <- W - U Sigma V.
// The matrix fits no cache, so what counts is how often it is streamed.  A product along the rows followed by one along
// the columns, q = W x and z = W^T q, needs ONE read: row i of W adds q_i W_i to z, and q_i = W_i x depends on that row
// alone, so a workgroup that holds a whole row in registers forms q_i and adds the row to its own z before it lets the
// row go (sk_pass_kernel).  A rank is it + 1 such passes.  The deflation is applied to the rows as they are read, with
// the same subtraction per element and in the same order as a stored update, and the matrix is written back only when
// no more pending u p^T fit in LDS.  Matrices of more than 32768 columns (a row does not fit a workgroup) take one
// stream per product instead, with the deflation stored once per rank.
// Q is renormalised after every power iteration (U, Sigma and V do not depend on the length of Q; the raw powers leave
// the fp32 range after a few iterations).  All sums have a fixed order: results are run-to-run identical.
#include "tq_device.h"

#include <algorithm>

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
// the matrix is read once per pass and fits no cache: the non-temporal hint on those loads is worth 8 % (measured)

__device__ inline float wave_sum(float v)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off);
    return v;
}

// y[i] = sum_j W'[i][j] x[j] with W' = W - u p^T written back when UPDATE.  One wave per row, four rows per workgroup
// and grid step.
template <bool UPDATE>
__global__ void __launch_bounds__(256) sk_rows_kernel(float* __restrict__ W, int64_t rows, int64_t cols,
                                                      const float* __restrict__ x, const float* __restrict__ u,
                                                      const float* __restrict__ p, float* __restrict__ y)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int64_t row = (int64_t)blockIdx.x * 4 + wave; row < rows; row += (int64_t)gridDim.x * 4) {
        float* wr = W + row * cols;
        const float ui = UPDATE ? u[row] : 0.f;
        float acc = 0.f;
        for (int64_t j = (int64_t)lane * 4; j < cols; j += 256) {
            // the update pass writes the row back in place, so it loads normally
            f32x4 w4 = UPDATE ? *reinterpret_cast<const f32x4*>(wr + j)
                              : __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(wr + j));
            if (UPDATE) {
                const f32x4 p4 = *reinterpret_cast<const f32x4*>(p + j);
                w4 -= ui * p4;
                *reinterpret_cast<f32x4*>(wr + j) = w4;
            }
            if (x) {
                const f32x4 x4 = *reinterpret_cast<const f32x4*>(x + j);
                acc = fmaf(w4[0], x4[0], acc); acc = fmaf(w4[1], x4[1], acc);
                acc = fmaf(w4[2], x4[2], acc); acc = fmaf(w4[3], x4[3], acc);
            }
        }
        acc = wave_sum(acc);
        if (lane == 0 && y) y[row] = acc;
    }
}

// partial[slab][j] = sum over the rows of the slab of W[i][j] q[i] * inv, inv = 1 / *norm (0 if the norm is 0) when a
// norm is given.  One thread per four columns; a row of a strip is one contiguous 4 KB read.
__global__ void __launch_bounds__(256) sk_cols_kernel(const float* __restrict__ W, int64_t rows, int64_t cols,
                                                      const float* __restrict__ q, const float* __restrict__ norm,
                                                      int64_t rows_per_slab, float* __restrict__ partial)
{
    const int64_t j = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
    const int64_t r0 = (int64_t)blockIdx.y * rows_per_slab;
    const int64_t r1 = r0 + rows_per_slab < rows ? r0 + rows_per_slab : rows;
    float inv = 1.f;
    if (norm) { const float n = *norm; inv = n > 0.f ? 1.f / n : 0.f; }
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    if (j < cols) {
        for (int64_t i = r0; i < r1; ++i) {
            const f32x4 w4 = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(W + i * cols + j));
            const float qi = q[i] * inv;
            acc += qi * w4;
        }
        *reinterpret_cast<f32x4*>(partial + (int64_t)blockIdx.y * cols + j) = acc;
    }
}

__global__ void __launch_bounds__(256) sk_colsum_kernel(const float* __restrict__ partial, int slabs, int64_t cols,
                                                        float* __restrict__ z)
{
    const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (j >= cols) return;
    float acc = 0.f;
    int s = 0;
    for (; s + 8 <= slabs; s += 8) {       // eight loads in flight, added in slab order
        float v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = partial[(int64_t)(s + i) * cols + j];
#pragma unroll
        for (int i = 0; i < 8; ++i) acc += v[i];
    }
    for (; s < slabs; ++s) acc += partial[(int64_t)s * cols + j];
    z[j] = acc;
}

// *out = |v| (one workgroup: per-thread strided sums in fp32, then a tree in LDS; fixed order)
__global__ void __launch_bounds__(1024) sk_norm_kernel(const float* __restrict__ v, int64_t n, float* __restrict__ out)
{
    __shared__ float red[1024];
    float acc = 0.f;
    for (int64_t i = threadIdx.x; i < n; i += 1024) acc = fmaf(v[i], v[i], acc);
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int s = 512; s >= 1; s >>= 1) {
        if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = sqrtf(red[0]);
}

// out[i] = v[i] / *norm (zeros if the norm is zero: the matrix has run out of rank); sigma_out = *norm * sigma_scale
__global__ void __launch_bounds__(256) sk_scale_kernel(const float* __restrict__ v, int64_t n, const float* __restrict__ norm,
                                                       float* __restrict__ out, float* __restrict__ sigma_out)
{
    const float nv = *norm;
    const float inv = nv > 0.f ? 1.f / nv : 0.f;
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) out[i] = v[i] * inv;
    if (sigma_out && i == 0) *sigma_out = nv;
}

// One stream over W: rows are read (with the npend pending deflations w -= u_k[i] p_k applied, and stored back with
// WRITE); with DOT, q[i] = w_i . x, partial[workgroup][j] = sum of q[i] w_ij over the workgroup's rows and
// ssq[workgroup] = sum of its q[i]^2.
// Bound by the HBM stream.  A thread owns NC float4 columns of every row, so x and the column sums stay in registers for
// the whole pass, and R rows are in work while the next R are in flight; one barrier per R rows (the dot products'
// reduction over the waves).  The workgroup is as wide as the row needs (256 to 1024 threads, 1024 threads per CU in all):
// registers hold at most 32768 columns (there x moves to LDS and the pending vector is read through the L2).
// Measured on 16384 x 12672 (831 MB): 130-136 us a pass = 6.1-6.4 TB/s with up to three pending deflations (295 us where it
// also stores), against 119 us for the product along the rows, 135 + 6 us for the one along the columns and 319 us for
// the stored deflation as passes of their own: rank 16 with two power iterations went from 16.6 to 7.8 ms.
template <int NT, int NC, int R, bool XLDS, bool DOT, bool WRITE>
__global__ void __launch_bounds__(NT, 4) sk_pass_kernel(float* __restrict__ W, int64_t rows, int64_t cols,
                                                     const float* __restrict__ x, const float* __restrict__ U0,
                                                     const float* __restrict__ P0, int npend, float* __restrict__ q,
                                                     float* __restrict__ partial, float* __restrict__ ssq)
{
    constexpr int NW = NT / 64;
    extern __shared__ __attribute__((aligned(16))) float sm[];      // red [2][R][NW] | x [cols] (XLDS) or p [npend][cols]
    float* red = sm;
    float* vec = sm + 2 * R * NW;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t G = gridDim.x, b = blockIdx.x;
    const int nsteps = (int)((rows - b * R + G * R - 1) / (G * R));      // groups of R rows: b, b + G, ...
    // columns past the end repeat the last four: they meet x = 0 and are never stored
    // (byte offsets next to a scalar row pointer, recomputed at each use: held or hoisted they would not fit the 128
    // registers that 1024 threads per CU leave)
    const uint32_t end = (uint32_t)cols * 4u;
    auto lane_off = [&]() {
        uint32_t o = (uint32_t)tid * 16u;
        asm volatile("" : "+v"(o));
        return o;
    };
    auto at = [&](uint32_t o, int c) { return min(o + (uint32_t)(c * NT * 16), end - 16u); };
    auto live = [&](uint32_t o, int c) { return o + (uint32_t)(c * NT * 16) < end; };
    auto f4 = [](const float* p, uint32_t o) { return reinterpret_cast<const f32x4*>(reinterpret_cast<const uint8_t*>(p) + o); };
    f32x4 xr[XLDS ? 1 : NC], acc[NC];
    if (DOT) {
        const uint32_t o = lane_off();
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            acc[c] = f32x4{0.f, 0.f, 0.f, 0.f};
            if constexpr (!XLDS) xr[c] = live(o, c) ? *f4(x, at(o, c)) : f32x4{0.f, 0.f, 0.f, 0.f};
        }
    }
    if (XLDS ? DOT : npend > 0) {
        const float* src = XLDS ? x : P0;
        const int64_t n = XLDS ? cols : npend * cols, n_pad = XLDS ? (int64_t)NC * NT * 4 : n;      // x is padded with zeros
        for (int64_t i = (int64_t)tid * 4; i < n_pad; i += NT * 4)
            *reinterpret_cast<f32x4*>(vec + i) = i < n ? *reinterpret_cast<const f32x4*>(src + i) : f32x4{0.f, 0.f, 0.f, 0.f};
        __syncthreads();
    }
    float sq = 0.f;
    auto row_of = [&](int s, int r) { return ((int64_t)s * G + b) * R + r; };
    auto load = [&](f32x4 (&w)[R][NC], int s) {      // rows past the end repeat the last one: they count with q = 0
        const uint32_t o = lane_off();
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int64_t i = row_of(s, r);
            const float* wr = W + (i < rows ? i : rows - 1) * cols;
#pragma unroll
            for (int c = 0; c < NC; ++c) w[r][c] = WRITE ? *f4(wr, at(o, c)) : __builtin_nontemporal_load(f4(wr, at(o, c)));
        }
    };
    auto work = [&](f32x4 (&w)[R][NC], int s) {
        const uint32_t o = lane_off();
        for (int k = 0; k < npend; ++k) {
            float ui[R];
#pragma unroll
            for (int r = 0; r < R; ++r) ui[r] = U0[k * rows + (row_of(s, r) < rows ? row_of(s, r) : rows - 1)];
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                const f32x4 p4 = *f4((XLDS ? P0 : vec) + k * cols, at(o, c));
#pragma unroll
                for (int r = 0; r < R; ++r) w[r][c] -= ui[r] * p4;
            }
        }
        if (WRITE) {
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (row_of(s, r) < rows) {
#pragma unroll
                    for (int c = 0; c < NC; ++c)
                        if (live(o, c)) *const_cast<f32x4*>(f4(W + row_of(s, r) * cols, at(o, c))) = w[r][c];
                }
        }
        if constexpr (DOT) {
            float* rd = red + (s & 1) * (R * NW);
#pragma unroll
            for (int r = 0; r < R; ++r) {
                float d = 0.f;
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    f32x4 x4;
                    if constexpr (XLDS) x4 = *f4(vec, o + (uint32_t)(c * NT * 16));
                    else x4 = xr[c];
#pragma unroll
                    for (int i = 0; i < 4; ++i) d = fmaf(w[r][c][i], x4[i], d);
                }
                d = wave_sum(d);
                if (lane == 0) rd[r * NW + wave] = d;
            }
            tqdev::lds_barrier();
#pragma unroll
            for (int r = 0; r < R; ++r) {
                float qv = 0.f;
#pragma unroll
                for (int i = 0; i < NW; i += 4) {
                    const f32x4 t = *reinterpret_cast<const f32x4*>(rd + r * NW + i);
                    qv += (t[0] + t[1]) + (t[2] + t[3]);
                }
                const bool in = row_of(s, r) < rows;
                if (tid == 0 && in) q[row_of(s, r)] = qv;
                qv = in ? qv : 0.f;
                sq = fmaf(qv, qv, sq);
#pragma unroll
                for (int c = 0; c < NC; ++c) acc[c] += qv * w[r][c];
            }
        }
    };
    f32x4 wa[R][NC], wb[R][NC];
    load(wa, 0);
    load(wb, 1);
    for (int s = 0; s < nsteps; s += 2) {
        work(wa, s);
        load(wa, s + 2);
        if (s + 1 < nsteps) work(wb, s + 1);
        load(wb, s + 3);
    }
    if (DOT) {
        const uint32_t o = lane_off();
#pragma unroll
        for (int c = 0; c < NC; ++c)
            if (live(o, c)) *const_cast<f32x4*>(f4(partial + b * cols, at(o, c))) = acc[c];
        if (tid == 0) ssq[b] = sq;
    }
}

// Ends a pass: z[j] = inv * sum of the G partial sums of column j, inv = 1 / |q| from the G partial sums of squares
// (0 if that is zero: the matrix has run out of rank); with u, u[i] = q[i] * inv as well.  Latency-bound: 64 columns per
// workgroup, the partial sums in 16 groups side by side; workgroups past the columns take their share of u.
__global__ void __launch_bounds__(256) sk_finish_kernel(const float* __restrict__ partial, int G, int64_t cols,
                                                        const float* __restrict__ ssq, float* __restrict__ z,
                                                        const float* __restrict__ q, int64_t rows, float* __restrict__ u)
{
    __shared__ f32x4 red[16][16];
    __shared__ float sred[256];
    const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
    const int64_t j = ((int64_t)blockIdx.x * 16 + tx) * 4;
    float sq = 0.f;
    for (int g = tid; g < G; g += 256) sq += ssq[g];
    sred[tid] = sq;
    f32x4 a = {0.f, 0.f, 0.f, 0.f};
    if (j < cols) {
        const int per = (G + 15) / 16, g1 = min(G, (ty + 1) * per);
        int g = ty * per;
        for (; g + 8 <= g1; g += 8) {
            f32x4 v[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = *reinterpret_cast<const f32x4*>(partial + (int64_t)(g + i) * cols + j);
#pragma unroll
            for (int i = 0; i < 8; ++i) a += v[i];
        }
        for (; g < g1; ++g) a += *reinterpret_cast<const f32x4*>(partial + (int64_t)g * cols + j);
    }
    red[ty][tx] = a;
    __syncthreads();
    for (int s = 128; s >= 1; s >>= 1) {
        if (tid < s) sred[tid] += sred[tid + s];
        __syncthreads();
    }
    const float n = sqrtf(sred[0]), inv = n > 0.f ? 1.f / n : 0.f;
    if (ty == 0 && j < cols) {
        for (int i = 1; i < 16; ++i) a += red[i][tx];
        *reinterpret_cast<f32x4*>(z + j) = a * inv;
    }
    if (u)
        for (int64_t i = (int64_t)blockIdx.x * 256 + tid; i < rows; i += (int64_t)gridDim.x * 256) u[i] = q[i] * inv;
}

// V[rho] (p = Sigma V on entry) becomes a unit vector, its length goes to sigma[rho]; one workgroup per rank
__global__ void __launch_bounds__(1024) sk_unit_kernel(float* __restrict__ V, int64_t cols, float* __restrict__ sigma)
{
    __shared__ float red[1024];
    float* v = V + (int64_t)blockIdx.x * cols;
    float acc = 0.f;
    for (int64_t i = threadIdx.x; i < cols; i += 1024) acc = fmaf(v[i], v[i], acc);
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int s = 512; s >= 1; s >>= 1) {
        if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
        __syncthreads();
    }
    const float n = sqrtf(red[0]), inv = n > 0.f ? 1.f / n : 0.f;
    for (int64_t i = threadIdx.x; i < cols; i += 1024) v[i] *= inv;
    if (threadIdx.x == 0) sigma[blockIdx.x] = n;
}

// Shape of the fused pass for a row length: threads, float4 columns per thread, rows in work at a time; workgroups and
// pending deflations that 156 KB of LDS per CU hold.  1024 threads per CU whatever the width.  Whole calls of rank 8 with two
// power iterations, a stream per product against this (us): 1024 x 1024 1384 / 255, 16384 x 1024 2021 / 686, 1024 x 2048
// 897 / 256, 2048 x 4096 905 / 669, 32768 x 4096 5542 / 3096, 1024 x 8192 919 / 641, 4096 x 8192 1705 / 1037, 4096 x 8196
// 1819 / 1024, 4096 x 16384 3034 / 1591, 4096 x 20000 3629 / 2269, 4096 x 32768 5644 / 3510, 16 x 32768 1273 / 360.  Matrices of so few
// rows that a workgroup has one group of them (2048 x 4096, 1024 x 8192) write a row of partial sums per group and gain least.
struct SketchShape {
    int nt, nc, rr, wg, maxpend;
    bool xlds;
};
bool sketch_shape(int64_t rows, int64_t cols, SketchShape* s)
{
    if (cols > 32768) return false;
    s->xlds = cols > 16384;
    s->nt = cols <= 4096 ? 256 : cols <= 8192 ? 512 : 1024;
    s->nc = cols <= 1024 ? 1 : cols <= 2048 ? 2 : cols <= 16384 ? 4 : 8;
    s->rr = s->xlds ? 1 : 8 / s->nc;
    const int per_cu = 1024 / s->nt;
    s->wg = (int)std::min<int64_t>(256 * per_cu, (rows + s->rr - 1) / s->rr);
    s->maxpend = s->xlds ? 1 : (int)std::min<int64_t>(4, 156 * 1024 / per_cu / (cols * 4));
    return true;
}

template <bool DOT, bool WRITE>
tq_status launch_pass(const SketchShape& s, float* W, int64_t rows, int64_t cols, const float* x, const float* U0,
                      const float* P0, int npend, float* q, float* partial, float* ssq, hipStream_t st)
{
    const size_t smem = ((size_t)2 * s.rr * (s.nt / 64) + (s.xlds ? (size_t)(DOT ? s.nc * s.nt * 4 : 0) : (size_t)npend * cols)) * 4;
#define TQ_SKP(NT, NC, R, XL)                                                                                            \
    hipLaunchKernelGGL((sk_pass_kernel<NT, NC, R, XL, DOT, WRITE>), dim3(s.wg), dim3(NT), smem, st, W, rows, cols, x, U0, P0, npend, \
                       q, partial, ssq)
    if (s.xlds) TQ_SKP(1024, 8, 1, true);
    else if (s.nc == 1) TQ_SKP(256, 1, 8, false);
    else if (s.nc == 2) TQ_SKP(256, 2, 4, false);
    else if (s.nt == 256) TQ_SKP(256, 4, 2, false);
    else if (s.nt == 512) TQ_SKP(512, 4, 2, false);
    else TQ_SKP(1024, 4, 2, false);
#undef TQ_SKP
    TQ_CHECK_LAUNCH();
    return TQ_OK;
}

struct SketchPlan {
    int slabs;
    int64_t rows_per_slab;
    size_t q, z, p, partial, norms, total;
    bool fused;
    SketchShape shape;
};

bool make_plan(int64_t rows, int64_t cols, SketchPlan* P)
{
    if (rows < 1 || cols < 4 || (cols & 3) || rows > (int64_t)1 << 24 || cols > (int64_t)1 << 24) return false;
    const int64_t strips = (cols / 4 + 255) / 256;
    int64_t slabs = (1024 + strips - 1) / strips;          // about 1024 workgroups per product along the columns
    if (slabs > rows) slabs = rows;
    if (slabs > 1024) slabs = 1024;
    if (slabs < 1) slabs = 1;
    P->rows_per_slab = (rows + slabs - 1) / slabs;
    P->slabs = (int)((rows + P->rows_per_slab - 1) / P->rows_per_slab);
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off += tq_align256(bytes); return o; };
    P->q = take((size_t)rows * 4);
    P->z = take((size_t)cols * 4);
    P->p = take((size_t)cols * 4);
    P->fused = sketch_shape(rows, cols, &P->shape);
    P->partial = take((size_t)(P->fused ? P->shape.wg : P->slabs) * cols * 4);
    P->norms = take(1024 * 4);          // fused pass: one sum of squares per workgroup
    P->total = off;
    return true;
}

}  // namespace

tq_status tqi_setup_sketch()
{
    bool ok = true;
#define TQ_ATTR1(NT, NC, R, XL, D, WR)                                                                                   \
    ok = ok && hipFuncSetAttribute((const void*)sk_pass_kernel<NT, NC, R, XL, D, WR>,                                    \
                                   hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024) == hipSuccess
#define TQ_ATTR(NT, NC, R, XL) TQ_ATTR1(NT, NC, R, XL, true, false); TQ_ATTR1(NT, NC, R, XL, true, true); TQ_ATTR1(NT, NC, R, XL, false, true)
    TQ_ATTR(1024, 8, 1, true);
    TQ_ATTR(512, 4, 2, false); TQ_ATTR(1024, 4, 2, false);
#undef TQ_ATTR
#undef TQ_ATTR1
    return ok ? TQ_OK : TQ_ERR_HIP;
}

extern "C" size_t tq_sketch_workspace_size(int64_t rows, int64_t cols)
{
    SketchPlan P;
    return make_plan(rows, cols, &P) ? P.total : 0;
}

extern "C" tq_status tq_sketch_lowrank(float* W, int64_t rows, int64_t cols, int32_t r, int32_t it, const float* sketch,
                                       float* U, float* sigma, float* V, void* workspace, size_t workspace_bytes,
                                       void* stream)
{
    if (!W || !sketch || !U || !sigma || !V || !workspace) return TQ_ERR_NULL;
    SketchPlan P;
    if (!make_plan(rows, cols, &P) || r < 1 || r > 4096 || it < 0 || it > 64) return TQ_ERR_SHAPE;
    if (((uintptr_t)W | (uintptr_t)sketch | (uintptr_t)V | (uintptr_t)workspace) & 15) return TQ_ERR_ALIGN;
    if (((uintptr_t)U | (uintptr_t)sigma) & 3) return TQ_ERR_ALIGN;
    if (workspace_bytes < P.total) return TQ_ERR_WORKSPACE;
    hipStream_t st = (hipStream_t)stream;
    uint8_t* ws = (uint8_t*)workspace;
    float* q = (float*)(ws + P.q);
    float* z = (float*)(ws + P.z);
    float* p = (float*)(ws + P.p);
    float* partial = (float*)(ws + P.partial);
    float* norms = (float*)(ws + P.norms);        // [0] |q|, [1] |p|; fused pass: sums of squares per workgroup
    if (P.fused) {
        const TqDeviceState* ds = nullptr;
        if (tqi_device_state(&ds) != TQ_OK) return TQ_ERR_HIP;      // (raised dynamic-LDS limits)
        const SketchShape& sh = P.shape;
        const unsigned fin = (unsigned)((cols + 63) / 64);
        // where u is written the grid covers the rows as well, 256 per workgroup: on the few workgroups that a narrow matrix has
        // columns for, u took longer than the passes (1000000 x 4, rank 4, no power iteration: 6.2 ms, now 2.5; 100000 x 64, rank 8:
        // 1304 us, now 566; 16384 x 1024 267, now 261)
        const unsigned fin_u = std::max(fin, (unsigned)std::min<int64_t>(1024, (rows + 255) / 256));
        int npend = 0;                 // the last npend deflations are not in W yet: u_k in U, p_k in V
        for (int rho = 0; rho < r; ++rho) {
            const float* x = sketch + (size_t)rho * cols;
            for (int i = 0; i <= it; ++i) {
                const float *U0 = U + (size_t)(rho - npend) * rows, *P0 = V + (size_t)(rho - npend) * cols;
                const bool write = i == 0 && npend == sh.maxpend;
                const tq_status rc = write ? launch_pass<true, true>(sh, W, rows, cols, x, U0, P0, npend, q, partial, norms, st)
                                           : launch_pass<true, false>(sh, W, rows, cols, x, U0, P0, npend, q, partial, norms, st);
                if (rc != TQ_OK) return rc;
                if (write) npend = 0;
                const bool last = i == it;      // p = W^T U = Sigma V, kept in V until sk_unit_kernel
                hipLaunchKernelGGL(sk_finish_kernel, dim3(last ? fin_u : fin), dim3(256), 0, st, (const float*)partial, sh.wg, cols, (const float*)norms,
                                   last ? V + (size_t)rho * cols : z, (const float*)q, rows, last ? U + (size_t)rho * rows : (float*)nullptr);
                x = z;
            }
            TQ_CHECK_LAUNCH();
            ++npend;
        }
        // the pending deflations: W holds the residual on return
        const tq_status rc = launch_pass<false, true>(sh, W, rows, cols, nullptr, U + (size_t)(r - npend) * rows,
                                                      V + (size_t)(r - npend) * cols, npend, nullptr, nullptr, nullptr, st);
        if (rc != TQ_OK) return rc;
        hipLaunchKernelGGL(sk_unit_kernel, dim3(r), dim3(1024), 0, st, V, cols, sigma);
        TQ_CHECK_LAUNCH();
        return TQ_OK;
    }
    const unsigned row_blocks = (unsigned)((rows + 3) / 4 < 8192 ? (rows + 3) / 4 : 8192);
    const dim3 col_grid((unsigned)((cols / 4 + 255) / 256), (unsigned)P.slabs);
    const unsigned col_blocks = (unsigned)((cols + 255) / 256), rowv_blocks = (unsigned)((rows + 255) / 256);
    auto cols_product = [&](const float* vec, const float* norm, float* out) {      // out = W^T (vec / norm)
        hipLaunchKernelGGL(sk_cols_kernel, col_grid, dim3(256), 0, st, (const float*)W, rows, cols, vec, norm, P.rows_per_slab,
                           partial);
        hipLaunchKernelGGL(sk_colsum_kernel, dim3(col_blocks), dim3(256), 0, st, (const float*)partial, P.slabs, cols, out);
    };
    for (int rho = 0; rho < r; ++rho) {
        const float* s = sketch + (size_t)rho * cols;
        // Q = W s, with the previous rank's deflation W -= u p^T applied on the way
        if (rho == 0)
            hipLaunchKernelGGL(sk_rows_kernel<false>, dim3(row_blocks), dim3(256), 0, st, W, rows, cols, s, (const float*)nullptr,
                               (const float*)nullptr, q);
        else
            hipLaunchKernelGGL(sk_rows_kernel<true>, dim3(row_blocks), dim3(256), 0, st, W, rows, cols, s,
                               (const float*)(U + (size_t)(rho - 1) * rows), (const float*)p, q);
        for (int i = 0; i < it; ++i) {       // Q <- W W^T Q / |Q|
            hipLaunchKernelGGL(sk_norm_kernel, dim3(1), dim3(1024), 0, st, (const float*)q, rows, norms);
            cols_product(q, norms, z);
            hipLaunchKernelGGL(sk_rows_kernel<false>, dim3(row_blocks), dim3(256), 0, st, W, rows, cols, (const float*)z,
                               (const float*)nullptr, (const float*)nullptr, q);
        }
        float* u = U + (size_t)rho * rows;
        hipLaunchKernelGGL(sk_norm_kernel, dim3(1), dim3(1024), 0, st, (const float*)q, rows, norms);
        hipLaunchKernelGGL(sk_scale_kernel, dim3(rowv_blocks), dim3(256), 0, st, (const float*)q, rows, (const float*)norms, u,
                           (float*)nullptr);
        // p = W^T U = Sigma V
        cols_product(u, nullptr, p);
        hipLaunchKernelGGL(sk_norm_kernel, dim3(1), dim3(1024), 0, st, (const float*)p, cols, norms + 1);
        hipLaunchKernelGGL(sk_scale_kernel, dim3(col_blocks), dim3(256), 0, st, (const float*)p, cols, (const float*)(norms + 1),
                           V + (size_t)rho * cols, sigma + rho);
        TQ_CHECK_LAUNCH();
    }
    // the last deflation: W holds the residual on return
    hipLaunchKernelGGL(sk_rows_kernel<true>, dim3(row_blocks), dim3(256), 0, st, W, rows, cols, (const float*)nullptr,
                       (const float*)(U + (size_t)(r - 1) * rows), (const float*)p, (float*)nullptr);
    TQ_CHECK_LAUNCH();
    return TQ_OK;
}
