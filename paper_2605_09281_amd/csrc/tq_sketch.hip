// Offline helper: rank-r approximation of a dense fp32 matrix by r Gaussian-sketch rank-1 deflations (Section 3.1,
// "Plug-in", Eq. 13), the replacement for the SVD of the tiled matrix W_big of Eq. 11.  Per rank, with sketch vector s:
//   Q = (W W^T)^it W s,   U = Q / |Q|,   Sigma = |Q^T W| / |Q|,   V = Q^T W / |Q^T W|,   W <- W - U Sigma V.
// The matrix fits no cache, so what counts is how often it is streamed, and it is not written until the end.  With u_j, p_j =
// W^T u_j of the ranks found so far (u_j orthonormal), the deflated matrix is never formed: W_k x = W x - sum_j u_j (p_j . x),
// and W_k^T W_k x = W^T q for q = W_k x.  A product along the rows followed by one along the columns needs ONE read: row i of
// W adds q_i W_i to z, and q_i = W_i x - sum_j u_ij (p_j . x) depends on that row alone, so a workgroup that holds a whole row in
// registers forms q_i and adds the row to its own z before it lets the row go (sk_pass_kernel).  The first product of every rank,
// W_k^T W_k s = W^T W s - sum_j p_j (p_j . s), comes out of ONE pair of block products for up to 16 ranks (Y = W S^T, Z = W^T Y on
// the 64-bit matrix instructions), so a rank is `it` passes more, not it + 1.  Vectors and sums are kept in 64 bits (u, p, q,
// z; the x of a pass is rounded to 32 bits, which changes nothing that follows: its p_j . x are formed from the rounded x): the
// subtractions cancel up to the square of Sigma_1 / Sigma_k, and q is made orthogonal to the u_j a second time after the pass
// (by d_j = u_j . q, formed in it), without which a rank past the last one would be noise inside the span of the others.
// After up to 16 ranks the residual is stored in one read and write, and the next ranks start from it.
// Matrices of more than 16384 columns take 32-bit column sums (registers) and therefore it + 1 passes; of more than 32768 (a row
// does not fit a workgroup) one stream per product, with the deflation stored once per rank.
// Q is renormalised after every power iteration (U, Sigma and V do not depend on the length of Q; the raw powers leave
// the fp32 range after a few iterations).  All sums have a fixed order: results are run-to-run identical.
#include "tq_device.h"

#include <algorithm>

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef double f64x4 __attribute__((ext_vector_type(4)));
constexpr int MAXB = 16;       // ranks between two stores of the residual (the N of the 64-bit matrix instruction)
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

// sum over the 16 lanes of a DPP row, in every lane
template <int CTRL>
__device__ inline double dpp_add(double v)
{
    const uint64_t b = __double_as_longlong(v);
    const uint32_t lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, 0xF, 0xF, true);
    const uint32_t hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), CTRL, 0xF, 0xF, true);
    return v + __longlong_as_double((int64_t)(((uint64_t)hi << 32) | lo));
}
__device__ inline double row_sum(double v)
{
    v = dpp_add<0xB1>(v);       // quad_perm 1,0,3,2
    v = dpp_add<0x4E>(v);       // quad_perm 2,3,0,1
    v = dpp_add<0x141>(v);      // row_half_mirror
    return dpp_add<0x140>(v);   // row_mirror
}
__device__ inline double wave_sum(double v)
{
    v = row_sum(v);
    v += __shfl_xor(v, 16);
    return v + __shfl_xor(v, 32);
}

constexpr int SK_CR(int nt) { return nt == 256 ? 1024 : 256; }      // rows between two visits of a pass to the u_ij

// One stream over W: q[i] = w_i . x - sum_{j<k} u_ij c_j with c_j = p_j . x (the sum of the n_c parts cpart[j cj + g cg]),
// partial[workgroup][j] = sum of q[i] w_ij over the workgroup's rows, ssq[workgroup] = sum of its q[i]^2 and
// dpart[workgroup][j] = sum of u_ij q[i].
// Bound by the HBM stream.  A thread owns NC float4 columns of every row, so the column sums stay in registers for the whole
// pass (x is in LDS), and R rows are in work while the next R are in flight; one barrier per R rows (the dot products' reduction
// over the waves).  The u_ij c_j of up to 256 rows (1024 on the
// narrow workgroups) are formed before them, the u_ij q_i after them.  The workgroup is as wide
// as the row needs (256 to 1024 threads, 1024 threads per CU in all): registers hold at most 16384 columns in 64 bits, 32768 in 32.
// Measured on 16384 x 12672 (831 MB): 135 us a pass = 6.1 TB/s.  Whole calls against passes that applied up to three stored deflations and
// kept everything in 32 bits: rank 16 with two power iterations 7.8 -> 5.4 ms, errors against 64 bits 1.0e-7 - 1.6e-7 -> 2.6e-8 (2-norms of
// the unit vectors, of which 2.5e-8 is the rounding of the results).  Three single rows in flight instead of two pairs: with 64-bit sums the
// pairs do not fit the registers.
template <int NT, int NC, int R, int NB, typename ACC>
__global__ void __launch_bounds__(NT, 4) sk_pass_kernel(const float* __restrict__ W, int64_t rows, int64_t cols,
                                                     const float* __restrict__ x, const double* __restrict__ U, int us, int k,
                                                     const double* __restrict__ cpart, int cj, int cg, int n_c, double* __restrict__ q,
                                                     ACC* __restrict__ partial, double* __restrict__ ssq, double* __restrict__ dpart)
{
    constexpr int NW = NT / 64, CR = SK_CR(NT), CS = CR / R;      // rows and steps between two visits to the u_ij
    typedef ACC acc4 __attribute__((ext_vector_type(4)));
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];      // red [16][MAXB] | coef [MAXB] | dsum [MAXB] | qs, qo [CR] | x [NC * NT * 4]
    double* red = reinterpret_cast<double*>(smem);
    double* coef = red + 16 * MAXB;
    double* dsum = coef + MAXB;
    double* qs = dsum + MAXB;
    double* qo = qs + CR;
    float* vec = reinterpret_cast<float*>(qo + CR);
    static_assert(2 * R * NW <= 16 * MAXB, "reduction buffer");
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
    auto row_of = [&](int s, int r) { return ((int64_t)s * G + b) * R + r; };
    auto load = [&](f32x4 (&w)[R][NC], int s) {      // rows past the end repeat the last one: they count with q = 0
        const uint32_t o = lane_off();
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const float* wr = W + min(row_of(s, r), rows - 1) * cols;
#pragma unroll
            for (int c = 0; c < NC; ++c) w[r][c] = __builtin_nontemporal_load(f4(wr, at(o, c)));
        }
    };
    f32x4 wq[NB][R][NC];
#pragma unroll
    for (int i = 0; i < NB; ++i) load(wq[i], i);
    const int uj = tid & (MAXB - 1), uc = uj < k ? uj : 0;
    auto u_at = [&](int s, int ci) { return U[min(row_of(s + ci / R, ci % R), rows - 1) * us + uc]; };
    double u0 = 0.;
    if (k > 0) {
        u0 = u_at(0, tid / MAXB);
        double c = 0.;
        for (int g = tid / MAXB; g < n_c; g += 4 * (NT / MAXB)) {      // four loads in flight
            double t[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) t[i] = cpart[(int64_t)uc * cj + (int64_t)min(g + i * (NT / MAXB), n_c - 1) * cg];
#pragma unroll
            for (int i = 0; i < 4; ++i) c += g + i * (NT / MAXB) < n_c ? t[i] : 0.;
        }
        c += __shfl_xor(c, 16);
        c += __shfl_xor(c, 32);
        if (lane < MAXB) red[wave * MAXB + lane] = c;
    }
    for (int64_t i = (int64_t)tid * 4; i < (int64_t)NC * NT * 4; i += NT * 4)
        *reinterpret_cast<f32x4*>(vec + i) = i < cols ? *reinterpret_cast<const f32x4*>(x + i) : f32x4{0.f, 0.f, 0.f, 0.f};
    double cf = 0.;
    if (k > 0) {
        __syncthreads();
#pragma unroll
        for (int w = 0; w < NW; ++w) cf += red[w * MAXB + uj];
        if (uj >= k) cf = 0.;
        if (tid < MAXB) { coef[tid] = cf; dsum[tid] = 0.; }
    }
    acc4 acc[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) acc[c] = acc4{0, 0, 0, 0};
    double sq = 0.;
    auto work = [&](const f32x4 (&w)[R][NC], int s, int s0) {
        const uint32_t o = lane_off();
        double* rd = red + (s & 1) * (R * NW);
        double d[R];
#pragma unroll
        for (int r = 0; r < R; ++r) d[r] = 0.;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const f32x4 x4 = *f4(vec, o + (uint32_t)(c * NT * 16));
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const double xd = x4[i];
#pragma unroll
                for (int r = 0; r < R; ++r) d[r] = fma((double)w[r][c][i], xd, d[r]);
            }
            __builtin_amdgcn_sched_barrier(0);      // (the conversions of a whole step at once would spill)
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            d[r] = wave_sum(d[r]);
            if (lane == 0) rd[r * NW + wave] = d[r];
        }
        tqdev::lds_barrier();
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int ci = (s - s0) * R + r;
            double qv = k > 0 ? -qs[ci] : 0.;
#pragma unroll
            for (int i = 0; i < NW; i += 2) {
                const f64x2 t = *reinterpret_cast<const f64x2*>(rd + r * NW + i);
                qv += t[0] + t[1];
            }
            qv = row_of(s, r) < rows ? qv : 0.;
            if (tid == 0) qo[ci] = qv;
            sq = fma(qv, qv, sq);
#pragma unroll
            for (int c = 0; c < NC; ++c)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    float e = w[r][c][i];
                    asm volatile("" : "+v"(e));      // converted again here: held from the dot product in 64 bits it would spill
                    acc[c][i] = fma((ACC)qv, (ACC)e, acc[c][i]);
                }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    for (int s0 = 0; s0 < nsteps; s0 += CS) {
        const int s1 = min(nsteps, s0 + CS);
        if (s0 > 0) {
#pragma unroll
            for (int i = 0; i < NB; ++i) load(wq[i], s0 + i);
        }
        __syncthreads();
        if (k > 0)
            for (int ci = tid / MAXB; ci < (s1 - s0) * R; ci += NT / MAXB) {
                const double c = row_sum((s0 == 0 && ci == tid / MAXB ? u0 : u_at(s0, ci)) * (s0 == 0 ? cf : coef[uj]));
                if (uj == 0) qs[ci] = c;
            }
        __syncthreads();
        for (int s = s0; s < s1; s += NB) {
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                if (s + i < s1) work(wq[i], s + i, s0);
                load(wq[i], s + i + NB);
            }
        }
        __syncthreads();
        for (int ci = tid; ci < (s1 - s0) * R; ci += NT) {
            const int64_t i = row_of(s0 + ci / R, ci % R);
            if (i < rows) q[i] = qo[ci];
        }
        if (k > 0) {
            double d = 0.;
            for (int ci = tid / MAXB; ci < (s1 - s0) * R; ci += NT / MAXB) {
                const int64_t i = row_of(s0 + ci / R, ci % R);
                if (uj < k && i < rows) d = fma(U[i * us + uj], qo[ci], d);
            }
            d += __shfl_xor(d, 16);
            d += __shfl_xor(d, 32);
            if (lane < MAXB) red[wave * MAXB + lane] = d;
            __syncthreads();
            if (tid < MAXB)
                for (int w = 0; w < NW; ++w) dsum[tid] += red[w * MAXB + tid];
        }
    }
    const uint32_t o = lane_off();
#pragma unroll
    for (int c = 0; c < NC; ++c)
        if (live(o, c))
            *reinterpret_cast<acc4*>(partial + b * cols + (o >> 2) + c * NT * 4) = acc[c];
    if (tid == 0) ssq[b] = sq;
    if (tid < k) dpart[b * MAXB + tid] = dsum[tid];
}

constexpr int FC = 32;      // columns per workgroup of the kernels between the passes (64 past 16384 columns: half as many parts for a pass to add up)

// The dot products that the next launch needs, of this workgroup's columns: 16 lanes for each vector m.  The operands are requested at
// the start of the kernel (load), the values v meet them at its end (store).
template <int FC>
struct SkDots {
    double a[FC / 16];
    template <typename T>
    __device__ void load(const T* p, int64_t j0, int64_t cols, int lo, int hi)
    {
        const int m = threadIdx.x >> 4, tx = threadIdx.x & 15;
        const bool in = m >= lo && m < hi;
#pragma unroll
        for (int i = 0; i < FC / 16; ++i) {
            const int64_t j = j0 + tx + 16 * i;
            a[i] = in && j < cols ? (double)p[m * cols + j] : 0.;
        }
    }
    __device__ void store(const double* v, double* out, int mstride) const
    {
        const int m = threadIdx.x >> 4, tx = threadIdx.x & 15;
        double d = 0.;
#pragma unroll
        for (int i = 0; i < FC / 16; ++i) d = fma(a[i], v[tx + 16 * i], d);
        d = row_sum(d);
        if (tx == 0) out[(int64_t)m * mstride] = d;
    }
};

// red[j] = the sum of n values at part + j * jstride, stride apart, for j < k; 0 for k <= j < 16.  256 threads, 16 for each j.
__device__ inline void sk_coefs(const double* part, int64_t jstride, int n, int stride, int k, double* red)
{
    const int tid = threadIdx.x, j = tid >> 4, tx = tid & 15;
    double c = 0.;
    if (j < k) {
        const double* p = part + j * jstride;
        int g = tx;
        for (; g + 112 < n; g += 128) {       // eight loads in flight
            double t[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) t[i] = p[(int64_t)(g + 16 * i) * stride];
#pragma unroll
            for (int i = 0; i < 8; ++i) c += t[i];
        }
        for (; g < n; g += 16) c += p[(int64_t)g * stride];
    }
    c = row_sum(c);
    if (tx == 0) red[j] = c;
}

// The first x of rank k from the block products: W_k^T W_k s = Z_k - sum_{j<k} p_j (p_j . s), scaled to the size of Z_k (a power of two),
// and its dot products with the p_j.  spart[j][m][workgroup] = parts of p_j . s_m; zexp[k][n_z]: exponents of Z_k.
__global__ void __launch_bounds__(256) sk_start_kernel(const double* __restrict__ Z, const int* __restrict__ zexp, int n_z, int64_t cols,
                                                       const double* __restrict__ P, int k, const double* __restrict__ spart,
                                                       float* __restrict__ x, double* __restrict__ cpart)
{
    __shared__ double v[FC], red[MAXB];
    __shared__ int ex[4];
    const int tid = threadIdx.x, n_c = gridDim.x;
    const int64_t j0 = (int64_t)blockIdx.x * FC, col = j0 + (tid & (FC - 1)), cl = min(col, cols - 1);
    SkDots<FC> dots;
    dots.load(P, j0, cols, 0, k);
    double a = Z[k * cols + cl], pj[MAXB];
#pragma unroll
    for (int j = 0; j < MAXB; ++j) {
        const double t = P[(j < k ? j : 0) * cols + cl];
        pj[j] = j < k ? t : 0.;
    }
    sk_coefs(spart + (int64_t)k * n_c, (int64_t)MAXB * n_c, n_c, 1, k, red);
    int e = -4096;
    for (int g = tid; g < n_z; g += 256) e = max(e, zexp[k * n_z + g]);
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) e = max(e, __shfl_xor(e, o));
    if ((tid & 63) == 0) ex[tid >> 6] = e;
    __syncthreads();
    if (tid < FC) {
#pragma unroll
        for (int j = 0; j < MAXB; ++j) a = fma(-pj[j], red[j], a);
        const float f = (float)ldexp(a, -max(max(ex[0], ex[1]), max(ex[2], ex[3])));
        if (col < cols) x[col] = f;
        v[tid] = col < cols ? (double)f : 0.;
    }
    __syncthreads();
    dots.store(v, cpart + (int64_t)blockIdx.x * MAXB, 1);
}

// Without power iterations: q = W_k s = Y_k - sum_{j<k} u_j c_j, c_j = p_j . s (also written to ctot), with the sums that a pass forms
__global__ void __launch_bounds__(256) sk_project_kernel(const double* __restrict__ Y, int us, int64_t rows,
                                                         const double* __restrict__ U, int k, const double* __restrict__ spart,
                                                         int n_c, double* __restrict__ q, double* __restrict__ ctot,
                                                         double* __restrict__ ssq, double* __restrict__ dpart)
{
    __shared__ double red[MAXB], sums[4][MAXB + 1];
    const int tid = threadIdx.x;
    sk_coefs(spart + (int64_t)k * n_c, (int64_t)MAXB * n_c, n_c, 1, k, red);
    __syncthreads();
    if (blockIdx.x == 0 && tid < MAXB) ctot[tid] = red[tid];
    double sq = 0., d[MAXB];
#pragma unroll
    for (int j = 0; j < MAXB; ++j) d[j] = 0.;
    for (int64_t i = (int64_t)blockIdx.x * 256 + tid; i < rows; i += (int64_t)gridDim.x * 256) {
        double u[MAXB], a = Y[i * us + k];
#pragma unroll
        for (int j = 0; j < MAXB; ++j) u[j] = U[i * us + (j < k ? j : 0)];
#pragma unroll
        for (int j = 0; j < MAXB; ++j) {
            if (j >= k) u[j] = 0.;
            a = fma(-u[j], red[j], a);
        }
        q[i] = a;
        sq = fma(a, a, sq);
#pragma unroll
        for (int j = 0; j < MAXB; ++j) d[j] = fma(u[j], a, d[j]);
    }
    sq = wave_sum(sq);
#pragma unroll
    for (int j = 0; j < MAXB; ++j) d[j] = wave_sum(d[j]);
    if ((tid & 63) == 0) {
        sums[tid >> 6][MAXB] = sq;
#pragma unroll
        for (int j = 0; j < MAXB; ++j) sums[tid >> 6][j] = d[j];
    }
    __syncthreads();
    if (tid <= MAXB) {
        const double t = (sums[0][tid] + sums[1][tid]) + (sums[2][tid] + sums[3][tid]);
        if (tid == MAXB) ssq[blockIdx.x] = t;
        else if (tid < k) dpart[(int64_t)blockIdx.x * MAXB + tid] = t;
    }
}

// Ends a pass: z = sum of the G partial sums, and q and z without what is left of the u_j in q (d_j, from the G_q parts; ce_j: parts of
// c_j that z does not account for yet), divided by |q| (0 where nothing is left: the matrix has run out of rank).  Then either x = z
// and its dot products with the p_j, or (LAST) u_k = q, p_k = z and the dot products of p_k with the sketch vectors to come.
// Latency-bound: 32 columns per workgroup, the partial sums in 32 groups side by side; the rows are shared out over all workgroups.
template <bool LAST, typename ACC>
__global__ void __launch_bounds__(256) sk_finish_kernel(const ACC* __restrict__ partial, int G, int G_q, int64_t cols, int n_c,
                                                        const double* __restrict__ ssq, const double* __restrict__ dpart,
                                                        const double* __restrict__ ce, double* __restrict__ P, int k, int nb,
                                                        float* __restrict__ x, double* __restrict__ cpart,
                                                        const double* __restrict__ q, int64_t rows, double* __restrict__ U, int us,
                                                        float* __restrict__ u_out, const float* __restrict__ S,
                                                        double* __restrict__ spart)
{
    typedef ACC acc4 __attribute__((ext_vector_type(4)));
    constexpr int FCN = sizeof(ACC) == 4 ? 2 * FC : FC, TX = FCN / 4, TY = 256 / TX;
    __shared__ double red[TY][FCN], dj[MAXB], de[MAXB], sred[4], v[FCN];
    const int tid = threadIdx.x, tx = tid % TX, ty = tid / TX;
    const int64_t j0 = (int64_t)blockIdx.x * FCN, j = j0 + tx * 4;
    const bool has_cols = (int)blockIdx.x < n_c;
    // everything that does not depend on the sums is requested first
    SkDots<FCN> dots;
    const int64_t col = j0 + (tid & (FCN - 1)), cl = min(col, cols - 1), row0 = (int64_t)blockIdx.x * 256 + tid;
    double pj[MAXB], uj[MAXB];
    if (has_cols) {
        if (LAST) dots.load(S, j0, cols, k + 1, nb);
        else dots.load(P, j0, cols, 0, k);
#pragma unroll
        for (int i = 0; i < MAXB; ++i) {
            const double t = P[(i < k ? i : 0) * cols + cl];
            pj[i] = i < k ? t : 0.;
        }
    }
    double qi = 0.;
    auto load_u = [&](int64_t i) {
        i = min(i, rows - 1);
        qi = q[i];
#pragma unroll
        for (int m = 0; m < MAXB; ++m) {
            const double t = U[i * us + (m < k ? m : 0)];
            uj[m] = m < k ? t : 0.;
        }
    };
    if (LAST) load_u(row0);
    double sq = 0.;
    for (int g = tid; g < G_q; g += 256) sq += ssq[g];
    sq = wave_sum(sq);
    if ((tid & 63) == 0) sred[tid >> 6] = sq;
    sk_coefs(dpart, 1, G_q, MAXB, k, dj);
    if (tid < MAXB) de[tid] = ce ? ce[tid] : 0.;
    if (has_cols) {
        f64x4 a = {0., 0., 0., 0.};
        if (j < cols) {
            const int per = (G + TY - 1) / TY, g1 = min(G, (ty + 1) * per);
            int g = ty * per;
            for (; g + 8 <= g1; g += 8) {
                acc4 t[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) t[i] = *reinterpret_cast<const acc4*>(partial + (int64_t)(g + i) * cols + j);
#pragma unroll
                for (int i = 0; i < 8; ++i)
#pragma unroll
                    for (int e = 0; e < 4; ++e) a[e] += (double)t[i][e];
            }
            for (; g < g1; ++g) {
                const acc4 t = *reinterpret_cast<const acc4*>(partial + (int64_t)g * cols + j);
#pragma unroll
                for (int e = 0; e < 4; ++e) a[e] += (double)t[e];
            }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) red[ty][tx * 4 + e] = a[e];
    }
    __syncthreads();
    sq = (sred[0] + sred[1]) + (sred[2] + sred[3]);
    double n2 = sq;
#pragma unroll
    for (int i = 0; i < MAXB; ++i) n2 -= dj[i] * dj[i];
    // below 1e-4 of its length q is the rounding of the first projection
    const double inv = n2 > 1e-8 * sq ? 1. / sqrt(n2) : 0.;
    if (has_cols) {
        if (tid < FCN) {
            double a = 0.;
#pragma unroll
            for (int i = 0; i < TY; ++i) a += red[i][tid];
#pragma unroll
            for (int i = 0; i < MAXB; ++i) a = fma(-pj[i], dj[i] + de[i], a);
            a *= inv;
            if (col >= cols) a = 0.;
            else if (LAST) P[k * cols + col] = a;
            else x[col] = (float)a;
            v[tid] = LAST ? a : (double)(float)a;
        }
        __syncthreads();
        if (LAST) dots.store(v, spart + (int64_t)k * MAXB * n_c + blockIdx.x, n_c);
        else dots.store(v, cpart + (int64_t)blockIdx.x * MAXB, 1);
    }
    if (LAST)
        for (int64_t i = row0; i < rows; i += (int64_t)gridDim.x * 256) {
            if (i != row0) load_u(i);
            double a = qi;
#pragma unroll
            for (int m = 0; m < MAXB; ++m) a = fma(-uj[m], dj[m], a);
            a *= inv;
            U[i * us + k] = a;
            u_out[i] = (float)a;
        }
}

// Y = W S^T for nb <= 16 sketch vectors, in 64 bits: Y[K-split][row][us].  v_mfma_f64_16x16x4: lane l holds row (column) l % 16 and
// index l / 16 of the contraction; here index i of step t is column 4 i + t of a group of 16, so that a lane's operands of four steps
// are one 16-byte load on either side.  32 rows per workgroup, whose eight waves share out the columns in runs of 64: two
// workgroups per CU, 8 KB of the matrix in flight per wave.
// Measured on 16384 x 12672, rank 16: 222 us (the rows of a lane group are 256 bytes apart pieces of 16 lines) and 170 for the columns,
// against 16 passes of 135 + 9.
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4, 4))) sk_block_rows_kernel(const float* __restrict__ W, int64_t rows, int64_t cols,
                                                               const float* __restrict__ S, int nb, int us, double* __restrict__ Y)
{
    __shared__ double red[8][2][16][17];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, rl = lane & 15, kq = lane >> 4;
    const int64_t r0 = (int64_t)blockIdx.x * 32;
    const int64_t step = (int64_t)gridDim.y * 8 * 64;
    const float* wr[2];
#pragma unroll
    for (int m = 0; m < 2; ++m) wr[m] = W + min(r0 + 16 * m + rl, rows - 1) * cols;
    const float* sr = S + (int64_t)(rl < nb ? rl : 0) * cols;
    f64x4 acc[2] = {{0., 0., 0., 0.}, {0., 0., 0., 0.}};
    struct Tile { f32x4 w[2][4], s[4]; };
    auto load = [&](Tile& t, int64_t c) {
#pragma unroll
        for (int h = 0; h < 4; ++h) {
            const int64_t col = min(c + 16 * h + 4 * kq, cols - 4);
#pragma unroll
            for (int m = 0; m < 2; ++m) t.w[m][h] = *reinterpret_cast<const f32x4*>(wr[m] + col);
            t.s[h] = *reinterpret_cast<const f32x4*>(sr + col);
        }
    };
    auto work = [&](const Tile& t, int64_t c) {
#pragma unroll
        for (int h = 0; h < 4; ++h) {
            const bool in = rl < nb && c + 16 * h + 4 * kq < cols;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const double b = in ? (double)t.s[h][i] : 0.;
#pragma unroll
                for (int m = 0; m < 2; ++m) acc[m] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)t.w[m][h][i], b, acc[m], 0, 0, 0);
            }
        }
    };
    int64_t c = ((int64_t)blockIdx.y * 8 + wave) * 64;
    Tile ta, tb;
    load(ta, c);
    load(tb, c + step);
    for (; c < cols; c += 2 * step) {
        work(ta, c);
        load(ta, c + 2 * step);
        work(tb, c + step);
        load(tb, c + 3 * step);
    }
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int i = 0; i < 4; ++i) red[wave][m][4 * i + kq][rl] = acc[m][i];      // D: row 4 i + lane / 16, column lane % 16
    __syncthreads();
    const int n = tid & 15, row = tid >> 4;
    double a = 0.;
#pragma unroll
    for (int w = 0; w < 8; ++w) a += red[w][row >> 4][row & 15][n];
    if (n < nb && r0 + row < rows) Y[((int64_t)blockIdx.y * rows + r0 + row) * us + n] = a;
}

// Z[slab][n][col] = sum over the slab's rows of Y[row][n] W[row][col]: the same instruction with the rows as the contraction; a wave owns
// 64 columns (four column tiles: column 4 (l % 16) + t of tile t, one 16-byte load) and a quarter of the slab's rows.
__global__ void __launch_bounds__(256, 4) sk_block_cols_kernel(const float* __restrict__ W, int64_t rows, int64_t cols,
                                                               const double* __restrict__ Y, int nb, int us, int64_t rows_per_slab,
                                                               double* __restrict__ Z)
{
    __shared__ double red[4][4][4][64];      // [wave][tile][register][lane]
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, rl = lane & 15, kq = lane >> 4;
    const int64_t c0 = (int64_t)blockIdx.x * 64 + 4 * rl, col = min(c0, cols - 4);
    const int64_t q4 = rows_per_slab / 4, r0 = blockIdx.y * rows_per_slab + wave * q4, r1 = min(r0 + q4, rows);
    const int n = rl < nb ? rl : 0;
    f64x4 acc[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) acc[t] = f64x4{0., 0., 0., 0.};
    constexpr int UN = 4;       // groups of four rows in work, and as many in flight
    struct Tile { f32x4 w[UN]; double y[UN]; };
    auto load = [&](Tile& t, int64_t r) {
#pragma unroll
        for (int g = 0; g < UN; ++g) {
            const int64_t row = min(r + 4 * g + kq, rows - 1);
            t.w[g] = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(W + row * cols + col));
            t.y[g] = Y[row * us + n];
        }
    };
    auto work = [&](const Tile& t, int64_t r) {
#pragma unroll
        for (int g = 0; g < UN; ++g) {
            const double a = rl < nb && r + 4 * g + kq < r1 ? t.y[g] : 0.;
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[i] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, (double)t.w[g][i], acc[i], 0, 0, 0);
        }
    };
    Tile ta, tb;
    load(ta, r0);
    load(tb, r0 + 4 * UN);
    for (int64_t r = r0; r < r1; r += 8 * UN) {
        work(ta, r);
        load(ta, r + 8 * UN);
        work(tb, r + 4 * UN);
        load(tb, r + 12 * UN);
    }
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) red[wave][t][i][lane] = acc[t][i];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int t = wave;      // this thread: tile `wave`, register i, its lane: rank 4 i + lane / 16, column 4 (lane % 16) + t
        const double a = (red[0][t][i][lane] + red[1][t][i][lane]) + (red[2][t][i][lane] + red[3][t][i][lane]);
        const int rank = 4 * i + kq;
        if (rank < nb && c0 + t < cols) Z[((int64_t)blockIdx.y * nb + rank) * cols + c0 + t] = a;
    }
}

// out[row][i] = sum of the n planes of `len` values per row (row: blockIdx.y), 64 values per workgroup; with zexp, the binary exponent of
// the largest of them (-4096: all zero)
__global__ void __launch_bounds__(256) sk_planes_kernel(const double* __restrict__ in, int n, int64_t len, double* __restrict__ out,
                                                        int* __restrict__ zexp)
{
    __shared__ double red[4][64];
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
    const int64_t plane = len * gridDim.y, i = (int64_t)blockIdx.x * 64 + tx, at = blockIdx.y * len + i;
    double a = 0.;
    if (i < len) {
        int p = ty;
        for (; p + 12 < n; p += 16) {
            double t[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) t[e] = in[(p + 4 * e) * plane + at];
            a += (t[0] + t[1]) + (t[2] + t[3]);
        }
        for (; p < n; p += 4) a += in[p * plane + at];
    }
    red[ty][tx] = a;
    __syncthreads();
    if (ty > 0) return;
    a = (red[0][tx] + red[1][tx]) + (red[2][tx] + red[3][tx]);
    if (i < len) out[at] = a;
    if (zexp) {       // (an infinity or a NaN scales by nothing that matters; the exponent stays inside what ldexp takes)
        int e = i < len && a != 0. ? min(max(ilogb(a), -1100), 1100) : -4096;
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) e = max(e, __shfl_xor(e, o));
        if (tx == 0) zexp[blockIdx.y * gridDim.x + blockIdx.x] = e;
    }
}

// W -= sum_{j<nb} u_j p_j^T, formed in 64 bits and rounded once.  A thread owns two columns of the p_j (16 x 2 in registers) and walks
// the slab's rows, eight in work and eight in flight; their u_j come from LDS, 64 rows at a time.
__global__ void __launch_bounds__(256, 3) sk_residual_kernel(float* __restrict__ W, int64_t rows, int64_t cols,
                                                             const double* __restrict__ U, int us, const double* __restrict__ P, int nb,
                                                             int64_t rows_per_slab)
{
    constexpr int UN = 8, CR = 64;
    __shared__ __attribute__((aligned(16))) double ul[CR][MAXB];
    const int tid = threadIdx.x;
    const int64_t j = min(((int64_t)blockIdx.x * 256 + tid) * 2, cols - 2);      // past the end: the last two again, not stored
    const bool in = ((int64_t)blockIdx.x * 256 + tid) * 2 < cols;
    const int64_t r0 = blockIdx.y * rows_per_slab, r1 = min(r0 + rows_per_slab, rows);
    f64x2 p[MAXB];
#pragma unroll
    for (int m = 0; m < MAXB; ++m) {
        const f64x2 t = *reinterpret_cast<const f64x2*>(P + (m < nb ? m : 0) * cols + j);
        p[m] = m < nb ? -t : f64x2{0., 0.};
    }
    auto load = [&](f32x2 (&w)[UN], int64_t i) {
#pragma unroll
        for (int e = 0; e < UN; ++e) w[e] = __builtin_nontemporal_load(reinterpret_cast<const f32x2*>(W + min(i + e, r1 - 1) * cols + j));
    };
    f32x2 wa[UN], wb[UN];
    load(wa, r0);
    for (int64_t c0 = r0; c0 < r1; c0 += CR) {
        __syncthreads();
        for (int i = tid; i < (int)min((int64_t)CR, (r1 - c0 + 2 * UN - 1) / (2 * UN) * (2 * UN)) * MAXB; i += 256) {
            const int64_t row = min(c0 + i / MAXB, r1 - 1);
            ul[i / MAXB][i % MAXB] = i % MAXB < nb ? U[row * us + i % MAXB] : 0.;
        }
        __syncthreads();
        auto work = [&](const f32x2 (&w)[UN], int o) {
#pragma unroll
            for (int e = 0; e < UN; ++e) {
                f64x2 a = {(double)w[e][0], (double)w[e][1]};
#pragma unroll
                for (int m = 0; m < MAXB; m += 2) {
                    const f64x2 u = *reinterpret_cast<const f64x2*>(&ul[o + e][m]);
                    a[0] = fma(u[1], p[m + 1][0], fma(u[0], p[m][0], a[0]));
                    a[1] = fma(u[1], p[m + 1][1], fma(u[0], p[m][1], a[1]));
                }
                if (in && c0 + o + e < r1) *reinterpret_cast<f32x2*>(W + (c0 + o + e) * cols + j) = f32x2{(float)a[0], (float)a[1]};
            }
        };
        const int n = (int)min((int64_t)CR, r1 - c0);
        for (int o = 0; o < n; o += 2 * UN) {
            load(wb, c0 + o + UN);
            work(wa, o);
            load(wa, c0 + o + 2 * UN);
            work(wb, o + UN);
        }
    }
}

// V[k] = p_k / |p_k|, sigma[k] = |p_k|; one workgroup per rank
__global__ void __launch_bounds__(1024) sk_unit_kernel(const double* __restrict__ P, int64_t cols, float* __restrict__ V,
                                                       float* __restrict__ sigma)
{
    __shared__ double red[16];
    const double* p = P + (int64_t)blockIdx.x * cols;
    float* v = V + (int64_t)blockIdx.x * cols;
    double acc = 0.;
    for (int64_t i = threadIdx.x; i < cols; i += 1024) acc = fma(p[i], p[i], acc);
    acc = wave_sum(acc);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
    __syncthreads();
    acc = 0.;
#pragma unroll
    for (int i = 0; i < 16; ++i) acc += red[i];
    const double n = sqrt(acc), inv = n > 0. ? 1. / n : 0.;
    for (int64_t i = threadIdx.x; i < cols; i += 1024) v[i] = (float)(p[i] * inv);
    if (threadIdx.x == 0) sigma[blockIdx.x] = (float)n;
}

// Shape of the fused pass for a row length: threads, float4 columns per thread, rows in work at a time; 1024 threads per CU
// whatever the width.
// Whole calls, deflations applied to the matrix in 32 bits against this, in us (rank, power iterations): 1024 x 1024
// (8, 2) 290 / 304, 1024 x 2048 (8, 2) 277 / 325, 2048 x 4096 (8, 2) 678 / 556, 1024 x 8192 (8, 2) 652 / 526, 32768 x 4096 (16, 1) 4302 / 2292,
// 4096 x 8192 (16, 2) 2055 / 1703, 4096 x 16384 (8, 2) 1616 / 1388, 6000 x 32768 (16, 1) 7416 / 5488, 100000 x 64 (8, 0) 582 / 262.  Matrices of a few MB
// wait for the launches in between, which carry longer chains of 64-bit sums.  At least four rows per workgroup: with one or two the partial
// sums are as many bytes as the matrix (2000 x 2400: 19 us a pass, 13.6 with four).
struct SketchShape {
    int nt, nc, rr, wg;
    bool wide;         // 32-bit column sums
};
bool sketch_shape(int64_t rows, int64_t cols, SketchShape* s)
{
    if (cols > 32768) return false;
    s->wide = cols > 16384;
    s->nt = cols <= 4096 ? 256 : cols <= 8192 ? 512 : 1024;
    s->nc = cols <= 1024 ? 1 : cols <= 2048 ? 2 : cols <= 16384 ? 4 : 8;
    s->rr = s->nc >= 4 ? 1 : 8 / s->nc;
    const int per_cu = 1024 / s->nt;
    const int64_t most = s->wide ? rows : (rows + 3) / 4;
    s->wg = (int)std::min<int64_t>(std::min<int64_t>(256 * per_cu, std::max<int64_t>(most, 1)), (rows + s->rr - 1) / s->rr);
    return true;
}

struct SketchPlan {
    int slabs;                      // unfused form
    int64_t rows_per_slab;
    size_t q, z, p, partial, norms;
    size_t total;
    bool fused;
    SketchShape shape;
    // fused form: ranks per batch, workgroups that finish a pass by columns, contraction splits and row slabs of the block
    // products and of the residual, workgroups of the projection without power iterations
    int nbs, n_c, ksplit, zslabs, wslabs, n_q;
    int64_t z_rows, w_rows;
    size_t x, U, P, Y, Z, cpart, spart, dpart, ssq, ctot, zexp;
};

bool make_plan(int64_t rows, int64_t cols, SketchPlan* P)
{
    if (rows < 1 || cols < 4 || (cols & 3) || rows > (int64_t)1 << 24 || cols > (int64_t)1 << 24) return false;
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off += tq_align256(bytes); return o; };
    auto cdiv = [](int64_t a, int64_t b) { return (a + b - 1) / b; };
    P->fused = sketch_shape(rows, cols, &P->shape);
    if (P->fused) {
        P->nbs = (int)std::min<int64_t>(MAXB, std::min(rows, cols));      // no batch has more ranks than the matrix
        P->n_c = (int)cdiv(cols, P->shape.wide ? 2 * FC : FC);
        P->n_q = (int)std::min<int64_t>(256, cdiv(rows, 256));
        // block products: two workgroups of 32 rows per CU; by columns four waves per SIMD
        P->ksplit = (int)std::max<int64_t>(1, std::min(512 / cdiv(rows, 32), cdiv(cols, 512)));
        P->zslabs = (int)std::max<int64_t>(1, std::min(1024 / cdiv(cols, 64), cdiv(rows, 64)));
        P->zslabs = std::min(P->zslabs, 256);
        P->z_rows = cdiv(cdiv(rows, P->zslabs), 16) * 16;
        P->zslabs = (int)cdiv(rows, P->z_rows);
        P->wslabs = (int)std::max<int64_t>(1, std::min(2048 / cdiv(cols, 512), cdiv(rows, 8)));
        P->w_rows = cdiv(rows, P->wslabs);
        P->wslabs = (int)cdiv(rows, P->w_rows);
        const size_t nb = P->nbs;
        P->q = take((size_t)rows * 8);
        P->x = take((size_t)cols * 4);
        P->U = take((size_t)rows * nb * 8);
        P->P = take((size_t)cols * nb * 8);
        P->Y = take((size_t)rows * nb * 8);
        P->Z = take((size_t)cols * nb * 8);
        const size_t pass = (size_t)P->shape.wg * cols * (P->shape.wide ? 4 : 8);
        const size_t yp = P->ksplit > 1 ? (size_t)P->ksplit * rows * nb * 8 : 0, zp = (size_t)P->zslabs * cols * nb * 8;
        P->partial = take(std::max(pass, std::max(yp, zp)));
        P->cpart = take((size_t)P->n_c * MAXB * 8);
        P->spart = take((size_t)P->n_c * MAXB * nb * 8);
        const size_t nq = std::max(P->shape.wg, P->n_q);
        P->dpart = take(nq * MAXB * 8);
        P->ssq = take(nq * 8);
        P->ctot = take(MAXB * 8);
        P->zexp = take((size_t)cdiv(cols, 64) * nb * 4);
        P->total = off;
        return true;
    }
    const int64_t strips = (cols / 4 + 255) / 256;
    int64_t slabs = (1024 + strips - 1) / strips;          // about 1024 workgroups per product along the columns
    if (slabs > rows) slabs = rows;
    if (slabs > 1024) slabs = 1024;
    if (slabs < 1) slabs = 1;
    P->rows_per_slab = (rows + slabs - 1) / slabs;
    P->slabs = (int)((rows + P->rows_per_slab - 1) / P->rows_per_slab);
    P->q = take((size_t)rows * 4);
    P->z = take((size_t)cols * 4);
    P->p = take((size_t)cols * 4);
    P->partial = take((size_t)P->slabs * cols * 4);
    P->norms = take(256);
    P->total = off;
    return true;
}

template <typename ACC>
tq_status fused_lowrank(const SketchPlan& P, float* W, int64_t rows, int64_t cols, int r, int it, const float* sketch, float* U_out,
                        float* sigma, float* V_out, uint8_t* ws, hipStream_t st)
{
    const SketchShape& sh = P.shape;
    auto f64 = [&](size_t o) { return reinterpret_cast<double*>(ws + o); };
    double *q = f64(P.q), *U = f64(P.U), *Pv = f64(P.P), *Y = f64(P.Y), *Z = f64(P.Z), *cpart = f64(P.cpart), *spart = f64(P.spart),
           *dpart = f64(P.dpart), *ssq = f64(P.ssq), *ctot = f64(P.ctot);
    float* x = reinterpret_cast<float*>(ws + P.x);
    int* zexp = reinterpret_cast<int*>(ws + P.zexp);
    ACC* partial = reinterpret_cast<ACC*>(ws + P.partial);
    const int us = P.nbs;
    const unsigned strips = (unsigned)((cols + 63) / 64);
    // where u is written the grid covers the rows as well, 256 per workgroup (a narrow matrix has few workgroups of columns)
    const unsigned fin_u = std::max((unsigned)P.n_c, (unsigned)std::min<int64_t>(1024, (rows + 255) / 256));
    const size_t smem = (size_t)(16 * MAXB + 2 * MAXB + 2 * SK_CR(sh.nt)) * 8 + (size_t)sh.nc * sh.nt * 16;
    auto pass = [&](int k, const float* xv, const double* parts, int cj, int cg) {
#define TQ_SKP(NT, NC, R, NB)                                                                                                  \
    hipLaunchKernelGGL((sk_pass_kernel<NT, NC, R, NB, ACC>), dim3(sh.wg), dim3(NT), smem, st, (const float*)W, rows, cols, xv, \
                       (const double*)U, us, k, parts, cj, cg, P.n_c, q, partial, ssq, dpart)
        if constexpr (sizeof(ACC) == 4) TQ_SKP(1024, 8, 1, 2);
        else if (sh.nc == 1) TQ_SKP(256, 1, 8, 2);
        else if (sh.nc == 2) TQ_SKP(256, 2, 4, 2);
        else if (sh.nt == 256) TQ_SKP(256, 4, 1, 3);
        else if (sh.nt == 512) TQ_SKP(512, 4, 1, 3);
        else TQ_SKP(1024, 4, 1, 3);
#undef TQ_SKP
    };
    for (int r0 = 0; r0 < r; r0 += P.nbs) {
        const int nb = std::min(P.nbs, r - r0);
        const float* S = sketch + (size_t)r0 * cols;
        // Two streams for the first products of the whole batch, against one per rank.  32-bit column sums do not bear the
        // cancellation of W^T W s.  Without power iterations the block saves a pass per rank but no launch, and takes four:
        // 1024 x 1024, rank 4: 92 us with, 83 without; 16384 x 1024, rank 16: 301 against 505 with passes alone.
        const bool block = sizeof(ACC) == 8 && nb >= 3 && (it > 0 || nb * rows * cols >= (int64_t)12 << 20);
        if (block) {
            double* parts = reinterpret_cast<double*>(ws + P.partial);
            hipLaunchKernelGGL(sk_block_rows_kernel, dim3((unsigned)((rows + 31) / 32), (unsigned)P.ksplit), dim3(512), 0, st, (const float*)W,
                               rows, cols, S, nb, us, P.ksplit > 1 ? parts : Y);
            if (P.ksplit > 1)
                hipLaunchKernelGGL(sk_planes_kernel, dim3((unsigned)((rows * us + 63) / 64)), dim3(256), 0, st, (const double*)parts, P.ksplit,
                                   rows * us, Y, (int*)nullptr);
            hipLaunchKernelGGL(sk_block_cols_kernel, dim3(strips, (unsigned)P.zslabs), dim3(256), 0, st, (const float*)W, rows, cols,
                               (const double*)Y, nb, us, P.z_rows, parts);
            hipLaunchKernelGGL(sk_planes_kernel, dim3(strips, nb), dim3(256), 0, st, (const double*)parts, P.zslabs, cols, Z, zexp);
            TQ_CHECK_LAUNCH();
        }
        for (int k = 0; k < nb; ++k) {
            auto finish = [&](bool last, const void* part, int G, int G_q, const double* ce) {
                if (last)
                    hipLaunchKernelGGL((sk_finish_kernel<true, ACC>), dim3(fin_u), dim3(256), 0, st, (const ACC*)part, G, G_q, cols, P.n_c,
                                       (const double*)ssq, (const double*)dpart, ce, Pv, k, nb, x, cpart, (const double*)q, rows, U, us,
                                       U_out + (size_t)(r0 + k) * rows, S, spart);
                else
                    hipLaunchKernelGGL((sk_finish_kernel<false, ACC>), dim3(P.n_c), dim3(256), 0, st, (const ACC*)part, G, G_q, cols, P.n_c,
                                       (const double*)ssq, (const double*)dpart, ce, Pv, k, nb, x, cpart, (const double*)q, rows, U, us,
                                       (float*)nullptr, S, spart);
            };
            if (block && it == 0) {
                hipLaunchKernelGGL(sk_project_kernel, dim3(P.n_q), dim3(256), 0, st, (const double*)Y, us, rows, (const double*)U, k,
                                   (const double*)spart, P.n_c, q, ctot, ssq, dpart);
                finish(true, Z + (size_t)k * cols, 1, P.n_q, ctot);
            } else {
                if (block)
                    hipLaunchKernelGGL(sk_start_kernel, dim3(P.n_c), dim3(256), 0, st, (const double*)Z, (const int*)zexp, (int)strips, cols,
                                       (const double*)Pv, k, (const double*)spart, x, cpart);
                for (int i = block ? 1 : 0; i <= it; ++i) {
                    if (i == 0) pass(k, S + (size_t)k * cols, (const double*)spart + (size_t)k * P.n_c, MAXB * P.n_c, 1);
                    else pass(k, x, cpart, 1, MAXB);
                    finish(i == it, partial, sh.wg, sh.wg, nullptr);
                }
            }
            TQ_CHECK_LAUNCH();
        }
        hipLaunchKernelGGL(sk_residual_kernel, dim3((unsigned)((cols + 511) / 512), (unsigned)P.wslabs), dim3(256), 0, st, W, rows, cols,
                           (const double*)U, us, (const double*)Pv, nb, P.w_rows);
        hipLaunchKernelGGL(sk_unit_kernel, dim3(nb), dim3(1024), 0, st, (const double*)Pv, cols, V_out + (size_t)r0 * cols, sigma + r0);
        TQ_CHECK_LAUNCH();
    }
    return TQ_OK;
}

}  // namespace

tq_status tqi_setup_sketch()
{
    // x of a pass takes up to 128 KB of LDS
    bool ok = true;
#define TQ_ATTR(NT, NC, R, NB, ACC)                                                                                          \
    ok = ok && hipFuncSetAttribute((const void*)sk_pass_kernel<NT, NC, R, NB, ACC>, hipFuncAttributeMaxDynamicSharedMemorySize, \
                                   160 * 1024) == hipSuccess
    TQ_ATTR(1024, 8, 1, 2, float);
    TQ_ATTR(1024, 4, 1, 3, double);
#undef TQ_ATTR
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
    if (P.fused) {
        const TqDeviceState* ds = nullptr;
        if (tqi_device_state(&ds) != TQ_OK) return TQ_ERR_HIP;      // (raised dynamic-LDS limits)
        return P.shape.wide ? fused_lowrank<float>(P, W, rows, cols, r, it, sketch, U, sigma, V, ws, st)
                            : fused_lowrank<double>(P, W, rows, cols, r, it, sketch, U, sigma, V, ws, st);
    }
    float* q = (float*)(ws + P.q);
    float* z = (float*)(ws + P.z);
    float* p = (float*)(ws + P.p);
    float* partial = (float*)(ws + P.partial);
    float* norms = (float*)(ws + P.norms);        // [0] |q|, [1] |p|
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
