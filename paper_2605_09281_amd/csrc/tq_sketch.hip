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
// the k sums that a workgroup leaves for the next launch are this far apart, a workgroup's beside each other: every workgroup of that launch
// reads them all (at 16 always they were a quarter of the time between the passes)
__host__ __device__ constexpr int sk_stride(int k) { return k <= 4 ? 4 : k <= 8 ? 8 : MAXB; }
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
// a + b after exchanging the upper half of a with the lower half of b, halves of the wave (32) or of every 32 lanes (16): what is left holds
// a's sums over the halves in the lower one, b's in the upper one
template <int N>
__device__ inline double swap_add(double a, double b)
{
    typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
    const uint64_t x = __double_as_longlong(a), y = __double_as_longlong(b);
    u32x2 lo, hi;
    if constexpr (N == 32) {
        lo = __builtin_amdgcn_permlane32_swap((uint32_t)x, (uint32_t)y, false, false);
        hi = __builtin_amdgcn_permlane32_swap((uint32_t)(x >> 32), (uint32_t)(y >> 32), false, false);
    } else {
        lo = __builtin_amdgcn_permlane16_swap((uint32_t)x, (uint32_t)y, false, false);
        hi = __builtin_amdgcn_permlane16_swap((uint32_t)(x >> 32), (uint32_t)(y >> 32), false, false);
    }
    return __longlong_as_double((int64_t)(((uint64_t)hi[0] << 32) | lo[0])) + __longlong_as_double((int64_t)(((uint64_t)hi[1] << 32) | lo[1]));
}
__device__ inline double cross_row_sum(double v)      // over the four rows of 16 lanes
{
    v = swap_add<16>(v, v);
    return swap_add<32>(v, v);
}
__device__ inline double wave_sum(double v) { return cross_row_sum(row_sum(v)); }

// the sums over the wave of d[0..R): lane l has that of d[l / (64 / R)].  The values halve at each exchange, so that eight take 34 instructions
// instead of 160 and none waits for LDS.
template <int R>
__device__ inline double wave_sums(const double (&d)[R])
{
    static_assert(R == 1 || R == 4 || R == 8, "rows at a time");
    if constexpr (R == 1) return wave_sum(d[0]);
    else if constexpr (R == 4) return row_sum(swap_add<16>(swap_add<32>(d[0], d[2]), swap_add<32>(d[1], d[3])));
    else {
        double e[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) e[i] = swap_add<32>(d[i], d[i + 4]);
        const double a = swap_add<16>(e[0], e[2]), b = swap_add<16>(e[1], e[3]);
        const bool up = threadIdx.x & 8;
        double v = up ? b : a;
        const uint64_t o = __double_as_longlong(up ? a : b);
        const uint32_t lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)o, 0x128, 0xF, 0xF, true);      // row_ror 8
        const uint32_t hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(o >> 32), 0x128, 0xF, 0xF, true);
        v += __longlong_as_double((int64_t)(((uint64_t)hi << 32) | lo));
        v = dpp_add<0xB1>(v);
        v = dpp_add<0x4E>(v);
        return dpp_add<0x141>(v);
    }
}

constexpr int SK_CR(int nt) { return nt == 256 ? 1024 : 256; }      // rows between two visits of a pass to the u_ij

// One stream over W: q[i] = w_i . x - sum_{j<k} u_ij c_j with c_j = p_j . x (the sum of the n_c parts cpart[j cj + g cg]),
// partial[workgroup][j] = sum of q[i] w_ij over the workgroup's rows, ssq[workgroup] = sum of its q[i]^2 and
// dpart[workgroup][j] = sum of u_ij q[i].
// Bound by the HBM stream.  A thread owns NC float4 columns of every row, so the column sums stay in registers for the whole
// pass (x is in LDS), and R rows are in work while the next are in flight; one barrier per R rows (the dot products' reduction
// over the waves).  The u_ij c_j of up to 256 rows (1024 on the narrow workgroups) are formed before them, the u_ij q_i after them.  The
// workgroup is as wide as the row needs (256 to 1024 threads, 1024 threads per CU in all): registers hold at most 16384 columns in 64 bits, 32768
// in 32.  Measured on 16384 x 12672 (831 MB): 131 us a pass = 6.3 TB/s; errors against 64 bits 2.6e-8 (2-norms of the unit vectors,
// of which 2.5e-8 is the rounding of the results).  Three single rows in flight instead of two pairs: with 64-bit sums the pairs do not
// fit the registers.
// On matrices of a few MB it is latency: what the first step waits for is requested before the rows and the barriers leave the rows in
// flight; the reduction takes no LDS; the first u_ij are kept; with FEW, where no workgroup has more than NB steps, nothing is requested that
// is not used.  1024 x 2048: 8.2 -> 7.0 us a pass; 1024 x 20000 30.4 -> 28.1; 1000000 x 4 502 -> 403;
// 16384 x 12672 134.5 -> 131.
template <int NT, int NC, int R, int NB, bool FEW, typename ACC>
__global__ void __launch_bounds__(NT, FEW && NT == 256 ? 2 : 4) sk_pass_kernel(const float* __restrict__ W, int64_t rows, int64_t cols,
                                                     const float* __restrict__ x, const double* __restrict__ U, int us, int k,
                                                     const double* __restrict__ cpart, int cj, int cg, int n_c, double* __restrict__ q,
                                                     ACC* __restrict__ partial, double* __restrict__ ssq, double* __restrict__ dpart)
{
    constexpr int NW = NT / 64, CR = SK_CR(NT), CS = CR / R;      // rows and steps between two visits to the u_ij
    typedef ACC acc4 __attribute__((ext_vector_type(4)));
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];      // red [16][MAXB] | coef [MAXB] | dsum [MAXB] | qs, qo [CR] | ul [NT] | x [NC * NT * 4]
    double* red = reinterpret_cast<double*>(smem);
    double* coef = red + 16 * MAXB;
    double* dsum = coef + MAXB;
    double* qs = dsum + MAXB;
    double* qo = qs + CR;
    double* ul = qo + CR;      // the first u_ij, for the end of the first visit
    float* vec = reinterpret_cast<float*>(ul + NT);
    static_assert(2 * R * NW <= 16 * MAXB && NW * MAXB <= CR, "reduction buffers");
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
    auto f4w = [](float* p, uint32_t o) { return reinterpret_cast<f32x4*>(reinterpret_cast<uint8_t*>(p) + o); };
    auto row_of = [&](int s, int r) { return ((int64_t)s * G + b) * R + r; };
    // rows past the end repeat the last one: they count with q = 0; steps past the end are requested all the same, so that the waits can
    // be counted, but from one line a load
    auto load = [&](f32x4 (&w)[R][NC], int s) {
        const uint32_t o = s < nsteps ? lane_off() : 0u;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const float* wr = W + min(row_of(s, r), rows - 1) * cols;
#pragma unroll
            for (int c = 0; c < NC; ++c) w[r][c] = __builtin_nontemporal_load(f4(wr, at(o, c)));
        }
    };
    // what the first step waits for is requested before the rows: loads return in order
    const int uj = tid & (MAXB - 1), uc = uj < k ? uj : 0;
    auto u_at = [&](int s, int ci) { return U[min(row_of(s + ci / R, ci % R), rows - 1) * us + uc]; };
    double u0 = 0., ct[4] = {0., 0., 0., 0.};
    const int ks = sk_stride(k), kj = tid & (ks - 1), kg = tid / ks, kn = NT / ks;      // parts of the c_j: ks sums side by side
    auto load_c = [&](int g) {      // four loads in flight
#pragma unroll
        for (int i = 0; i < 4; ++i) ct[i] = cpart[(int64_t)(kj < k ? kj : 0) * cj + (int64_t)min(g + i * kn, n_c - 1) * cg];
    };
    if (k > 0) {
        load_c(kg);
        u0 = u_at(0, tid / MAXB);
    }
    f32x4 xv[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) xv[c] = *f4(x, at((uint32_t)tid * 16u, c));
    f32x4 wq[NB][R][NC];
#pragma unroll
    for (int i = 0; i < NB - 1; ++i)
        if (!FEW || i == 0 || i < nsteps) load(wq[i], i);
#pragma unroll
    for (int c = 0; c < NC; ++c)
        *f4w(vec, (uint32_t)(tid + c * NT) * 16u) = live((uint32_t)tid * 16u, c) ? xv[c] : f32x4{0.f, 0.f, 0.f, 0.f};
    if (!FEW || NB - 1 < nsteps) load(wq[NB - 1], NB - 1);      // (here: before x is out of the way there are no registers for it)
    double cf = 0.;
    if (k > 0) {
        double c = 0.;
        for (int g = kg; g < n_c; g += 4 * kn) {
            if (g != kg) load_c(g);
#pragma unroll
            for (int i = 0; i < 4; ++i) c += g + i * kn < n_c ? ct[i] : 0.;
        }
        if (ks <= 4) c = dpp_add<0x124>(c);      // row_ror 4
        if (ks <= 8) c = dpp_add<0x128>(c);      // row_ror 8
        c = cross_row_sum(c);
        if (lane < MAXB) qo[wave * MAXB + lane] = c;      // (free until the first step has passed its barrier)
        tqdev::lds_barrier();
#pragma unroll
        for (int w = 0; w < NW; ++w) cf += qo[w * MAXB + uj];
        if (uj >= k) cf = 0.;
        if (tid < MAXB) { coef[tid] = cf; dsum[tid] = 0.; }
        ul[tid] = u0;
        for (int ci = tid / MAXB; ci < min(nsteps, CS) * R; ci += NT / MAXB) {
            const double v = row_sum((ci == tid / MAXB ? u0 : u_at(0, ci)) * cf);
            if (uj == 0) qs[ci] = v;
        }
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
        const double dw = wave_sums<R>(d);
        if (lane % (64 / R) == 0) rd[lane / (64 / R) * NW + wave] = dw;
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
    for (int s0 = 0; s0 < nsteps; s0 += CS) {      // (FEW: once)
        const int s1 = min(nsteps, s0 + CS);
        if (s0 > 0) {
#pragma unroll
            for (int i = 0; i < NB; ++i) load(wq[i], s0 + i);
            __syncthreads();
            if (k > 0)
                for (int ci = tid / MAXB; ci < (s1 - s0) * R; ci += NT / MAXB) {
                    const double v = row_sum(u_at(s0, ci) * coef[uj]);
                    if (uj == 0) qs[ci] = v;
                }
        }
        // (x is in LDS since the barrier above where there were c_j to add up; qs is read behind the barrier of the first step)
        if (k == 0) tqdev::lds_barrier();
        for (int s = s0; s < s1; s += NB) {
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                if (s + i < s1) work(wq[i], s + i, s0);
                if (!FEW) load(wq[i], s + i + NB);
            }
            if (FEW) break;
        }
        if (s1 == nsteps) {
            const uint32_t o = lane_off();
#pragma unroll
            for (int c = 0; c < NC; ++c)
                if (live(o, c))
                    *reinterpret_cast<acc4*>(partial + b * cols + (o >> 2) + c * NT * 4) = acc[c];
            if (tid == 0) ssq[b] = sq;
        }
        tqdev::lds_barrier();
        for (int ci = tid; ci < (s1 - s0) * R; ci += NT) {
            const int64_t i = row_of(s0 + ci / R, ci % R);
            if (i < rows) q[i] = qo[ci];
        }
        if (k > 0) {
            double d = 0.;
            for (int ci = tid / MAXB; ci < (s1 - s0) * R; ci += NT / MAXB) {
                const int64_t i = row_of(s0 + ci / R, ci % R);
                if (uj < k && i < rows) d = fma(s0 == 0 && ci == tid / MAXB ? ul[tid] : U[i * us + uj], qo[ci], d);
            }
            d = cross_row_sum(d);
            if (lane < MAXB) red[wave * MAXB + lane] = d;
            tqdev::lds_barrier();
            if (tid < MAXB) {
                double t = 0.;
#pragma unroll
                for (int w = 0; w < NW; ++w) t += red[w * MAXB + tid];
                dsum[tid] += t;
            }
        }
    }
    if (tid < k) dpart[b * ks + tid] = dsum[tid];
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
    __device__ void store(const double* v, double* out, int mstride, int n = MAXB) const      // n: of the 16 vectors, those that are wanted
    {
        const int m = threadIdx.x >> 4, tx = threadIdx.x & 15;
        double d = 0.;
#pragma unroll
        for (int i = 0; i < FC / 16; ++i) d = fma(a[i], v[tx + 16 * i], d);
        d = row_sum(d);
        if (tx == 0 && m < n) out[(int64_t)m * mstride] = d;
    }
};

// red[j] = the sum of n values at part + j * jstride, stride apart, for j < k; 0 for k <= j < 16.  256 threads, 16 for each j.  The first eight
// loads are requested where load is called.
struct SkCoefs {
    double t[8];
    __device__ void load(const double* part, int64_t jstride, int n, int stride, int k, int g0 = 0)
    {
        const int j = threadIdx.x >> 4, tx = threadIdx.x & 15;
        const double* p = part + (j < k ? j : 0) * jstride;
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if (i == 0 || g0 + 16 * i < n) t[i] = p[(int64_t)min(g0 + tx + 16 * i, n - 1) * stride];
    }
    __device__ void store(const double* part, int64_t jstride, int n, int stride, int k, double* red)
    {
        const int j = threadIdx.x >> 4, tx = threadIdx.x & 15;
        double c = 0.;
        for (int g = 0; g < n; g += 128) {
            if (g > 0) load(part, jstride, n, stride, k, g);
#pragma unroll
            for (int i = 0; i < 8; ++i) c += g + tx + 16 * i < n ? t[i] : 0.;
        }
        c = row_sum(j < k ? c : 0.);
        if (tx == 0) red[j] = c;
    }
};

// The first x of rank k from the block products: W_k^T W_k s = Z_k - sum_{j<k} p_j (p_j . s), scaled to the size of Z_k (a power of two),
// and its dot products with the p_j.  spart[j][m][workgroup] = parts of p_j . s_m; zexp[k][n_z]: exponents of Z_k.
template <int KP>
__global__ void __launch_bounds__(256) sk_start_kernel(const double* __restrict__ Z, const int* __restrict__ zexp, int n_z, int64_t cols,
                                                       const double* __restrict__ P, int k, const double* __restrict__ spart,
                                                       float* __restrict__ x, double* __restrict__ cpart)
{
    __shared__ double v[FC], red[MAXB];
    __shared__ int ex[4];
    const int tid = threadIdx.x, n_c = gridDim.x;
    const int64_t j0 = (int64_t)blockIdx.x * FC, col = j0 + (tid & (FC - 1)), cl = min(col, cols - 1);
    SkDots<FC> dots;
    SkCoefs coefs;
    int e = zexp[k * n_z + min(tid, n_z - 1)];
    if (KP > 0) coefs.load(spart + (int64_t)k * n_c, (int64_t)MAXB * n_c, n_c, 1, k);
    double a = 0., pj[KP > 0 ? KP : 1];
    if (tid < FC) {      // (the threads that fold them)
        a = Z[k * cols + cl];
#pragma unroll
        for (int j = 0; j < KP; ++j) {
            const double t = P[(j < k ? j : 0) * cols + cl];
            pj[j] = j < k ? t : 0.;
        }
    }
    if (KP > 0) {
        dots.load(P, j0, cols, 0, k);
        coefs.store(spart + (int64_t)k * n_c, (int64_t)MAXB * n_c, n_c, 1, k, red);
    }
    for (int g = tid + 256; g < n_z; g += 256) e = max(e, zexp[k * n_z + g]);
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) e = max(e, __shfl_xor(e, o));
    if ((tid & 63) == 0) ex[tid >> 6] = e;
    __syncthreads();
    if (tid < FC) {
#pragma unroll
        for (int j = 0; j < KP; ++j) a = fma(-pj[j], red[j], a);
        const float f = (float)ldexp(a, -max(max(ex[0], ex[1]), max(ex[2], ex[3])));
        if (col < cols) x[col] = f;
        v[tid] = col < cols ? (double)f : 0.;
    }
    if (KP == 0) return;
    __syncthreads();
    dots.store(v, cpart + (int64_t)blockIdx.x * KP, 1, KP);
}

// u[m] = the first KP values at p, for m < k (0 behind), in pairs: a lane's row of the u_ij is a line of its own, and requests count
template <int KP>
__device__ inline void sk_load_u(const double* __restrict__ p, int k, double (&u)[KP])
{
    typedef double f64x2u __attribute__((ext_vector_type(2), aligned(8)));
#pragma unroll
    for (int m = 0; m < KP; m += 2) {
        const f64x2u t = *reinterpret_cast<const f64x2u*>(p + (m < k ? m : 0));      // (m + 1 <= k: inside the row)
        u[m] = m < k ? t[0] : 0.;
        u[m + 1] = m + 1 < k ? t[1] : 0.;
    }
}

// Without power iterations: q = W_k s = Y_k - sum_{j<k} u_j c_j, c_j = p_j . s (also written to ctot), with the sums that a pass forms
template <int KP>
__global__ void __launch_bounds__(256) sk_project_kernel(const double* __restrict__ U, int us, int64_t rows, int k,
                                                         const double* __restrict__ spart,
                                                         int n_c, double* __restrict__ q, double* __restrict__ ctot,
                                                         double* __restrict__ ssq, double* __restrict__ dpart)
{
    __shared__ double red[MAXB], sums[4][MAXB + 1];
    const int tid = threadIdx.x;
    double u[KP > 0 ? KP : 1], y = 0.;
    auto load = [&](int64_t i) {
        i = min(i, rows - 1);
        y = U[i * us + k];      // (Y_k, until u_k takes its place)
        if constexpr (KP > 0) sk_load_u<KP>(U + i * us, k, u);
    };
    SkCoefs coefs;
    if (KP > 0) coefs.load(spart + (int64_t)k * n_c, (int64_t)MAXB * n_c, n_c, 1, k);
    const int64_t row0 = (int64_t)blockIdx.x * 256 + tid;
    load(row0);
    coefs.store(spart + (int64_t)k * n_c, (int64_t)MAXB * n_c, KP > 0 ? n_c : 0, 1, k, red);
    __syncthreads();
    if (blockIdx.x == 0 && tid < MAXB) ctot[tid] = red[tid];
    double sq = 0., d[KP > 0 ? KP : 1];
#pragma unroll
    for (int j = 0; j < KP; ++j) d[j] = 0.;
    for (int64_t i = row0; i < rows; i += (int64_t)gridDim.x * 256) {
        if (i != row0) load(i);
        double a = y;
#pragma unroll
        for (int j = 0; j < KP; ++j) a = fma(-u[j], red[j], a);
        q[i] = a;
        sq = fma(a, a, sq);
#pragma unroll
        for (int j = 0; j < KP; ++j) d[j] = fma(u[j], a, d[j]);
    }
    sq = wave_sum(sq);
#pragma unroll
    for (int j = 0; j < KP; ++j) d[j] = wave_sum(d[j]);
    if ((tid & 63) == 0) {
        sums[tid >> 6][MAXB] = sq;
#pragma unroll
        for (int j = 0; j < KP; ++j) sums[tid >> 6][j] = d[j];
    }
    __syncthreads();
    if (tid < k || tid == MAXB) {
        const double t = (sums[0][tid] + sums[1][tid]) + (sums[2][tid] + sums[3][tid]);
        if (tid == MAXB) ssq[blockIdx.x] = t;
        else dpart[(int64_t)blockIdx.x * KP + tid] = t;
    }
}

// Ends a pass: z = sum of the G partial sums, and q and z without what is left of the u_j in q (d_j, from the G_q parts; ce_j: parts of
// c_j that z does not account for yet), divided by |q| (0 where nothing is left: the matrix has run out of rank).  Then either x = z
// and its dot products with the p_j, or (LAST) u_k = q, p_k = z and the dot products of p_k with the sketch vectors to come.
// Latency-bound: 32 columns per workgroup, the partial sums in 32 groups side by side; the rows are shared out over all workgroups; everything
// is requested before anything is waited for, and only what the k earlier ranks need (KP: k rounded up to 4, 8 or 16).  1024 x 2048, rank 8: 5.7
// and 7.2 us (LAST) -> 4.5 and 4.8.
template <bool LAST, int KP, typename ACC>
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
    // all that this kernel reads is requested before the first sum waits (in that order: loads return in order)
    double uj[KP > 0 ? KP : 1], qi = 0.;
    const int64_t row0 = (int64_t)blockIdx.x * 256 + tid;
    auto load_u = [&](int64_t i) {
        i = min(i, rows - 1);
        qi = q[i];
        if constexpr (KP > 0) sk_load_u<KP>(U + i * us, k, uj);
    };
    if (LAST) load_u(row0);
    double sq = ssq[min(tid, G_q - 1)];
    SkCoefs coefs;
    if (KP > 0) coefs.load(dpart, 1, G_q, KP, k);
    const int per = (G + TY - 1) / TY, g0 = ty * per, g1 = min(G, g0 + per);
    acc4 part[8];
    auto load_part = [&](int g) {
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if (i == 0 || g - g0 + i < per) part[i] = *reinterpret_cast<const acc4*>(partial + (int64_t)min(g + i, G - 1) * cols + min(j, cols - 4));
    };
    SkDots<FCN> dots;
    const int64_t col = j0 + (tid & (FCN - 1)), cl = min(col, cols - 1);
    double pj[KP > 0 ? KP : 1];
    if (has_cols) {
        load_part(g0);
        if (tid < FCN)      // (the threads that fold them)
#pragma unroll
            for (int i = 0; i < KP; ++i) {
                const double t = P[(i < k ? i : 0) * cols + cl];
                pj[i] = i < k ? t : 0.;
            }
        if (LAST) dots.load(S, j0, cols, k + 1, nb);
        else if (KP > 0) dots.load(P, j0, cols, 0, k);
    }
    if (tid >= G_q) sq = 0.;
    for (int g = tid + 256; g < G_q; g += 256) sq += ssq[g];
    sq = wave_sum(sq);
    if ((tid & 63) == 0) sred[tid >> 6] = sq;
    if (KP > 0) coefs.store(dpart, 1, G_q, KP, k, dj);
    if (tid < MAXB) de[tid] = ce ? ce[tid] : 0.;
    if (has_cols) {
        f64x4 a = {0., 0., 0., 0.};
        for (int g = g0; g < g1; g += 8) {
            if (g > g0) load_part(g);
#pragma unroll
            for (int i = 0; i < 8; ++i)
                if (i == 0 || g - g0 + i < per)
#pragma unroll
                    for (int e = 0; e < 4; ++e) a[e] += g + i < g1 ? (double)part[i][e] : 0.;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) red[ty][tx * 4 + e] = a[e];
    }
    __syncthreads();
    sq = (sred[0] + sred[1]) + (sred[2] + sred[3]);
    double n2 = sq;
#pragma unroll
    for (int i = 0; i < KP; ++i) n2 -= dj[i] * dj[i];
    // below 1e-4 of its length q is the rounding of the first projection
    const double inv = n2 > 1e-8 * sq ? 1. / sqrt(n2) : 0.;
    if (has_cols) {
        if (tid < FCN) {
            double a = 0.;
#pragma unroll
            for (int i = 0; i < TY; ++i) a += red[i][tid];
#pragma unroll
            for (int i = 0; i < KP; ++i) a = fma(-pj[i], dj[i] + de[i], a);
            a *= inv;
            // 32-bit column sums: x of about unit length instead of Sigma, as a power of two (the next sums have the size of Sigma^2 then, and
            // not of Sigma^3, which leaves the fp32 range for matrices of 1e12 or 1e-15)
            if (sizeof(ACC) == 4 && !LAST && inv > 0.) a = ldexp(a, ilogb(inv));
            if (col >= cols) a = 0.;
            else if (LAST) P[k * cols + col] = a;
            else x[col] = (float)a;
            v[tid] = LAST ? a : (double)(float)a;
        }
        if (LAST || KP > 0) {
            __syncthreads();
            if (LAST) dots.store(v, spart + (int64_t)k * MAXB * n_c + blockIdx.x, n_c);
            else dots.store(v, cpart + (int64_t)blockIdx.x * KP, 1, KP);
        }
    }
    if (LAST)
        for (int64_t i = row0; i < rows; i += (int64_t)gridDim.x * 256) {
            if (i != row0) load_u(i);
            double a = qi;
#pragma unroll
            for (int m = 0; m < KP; ++m) a = fma(-uj[m], dj[m], a);
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

// v = p / |p|, sigma = |p|, by one workgroup of 256
__device__ inline void sk_unit(const double* __restrict__ p, int64_t cols, float* __restrict__ v, float* __restrict__ sigma)
{
    __shared__ double red[4];
    const int tid = threadIdx.x;
    constexpr int NV = 8;       // four columns a thread, eight times in flight
    f64x4 t[NV];
    auto load = [&](int64_t j0) {
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int64_t j = j0 + ((int64_t)i * 256 + tid) * 4;
            if (i == 0 || j0 + (int64_t)i * 1024 < cols) t[i] = *reinterpret_cast<const f64x4*>(p + min(j, cols - 4));
        }
    };
    double acc = 0.;
    for (int64_t j0 = 0; j0 < cols; j0 += NV * 1024) {
        load(j0);
#pragma unroll
        for (int i = 0; i < NV; ++i)
            if (j0 + ((int64_t)i * 256 + tid) * 4 < cols)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc = fma(t[i][e], t[i][e], acc);
    }
    acc = wave_sum(acc);
    if ((tid & 63) == 0) red[tid >> 6] = acc;
    __syncthreads();
    const double n = sqrt((red[0] + red[1]) + (red[2] + red[3])), inv = n > 0. ? 1. / n : 0.;
    for (int64_t j0 = 0; j0 < cols; j0 += NV * 1024) {
        if (cols > NV * 1024) load(j0);
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int64_t j = j0 + ((int64_t)i * 256 + tid) * 4;
            if (j < cols) *reinterpret_cast<f32x4*>(v + j) = f32x4{(float)(t[i][0] * inv), (float)(t[i][1] * inv), (float)(t[i][2] * inv), (float)(t[i][3] * inv)};
        }
    }
    if (tid == 0) *sigma = (float)n;
}

// W -= sum_{j<nb} u_j p_j^T, formed in 64 bits and rounded once.  A thread owns two columns of the p_j (16 x 2 in registers) and walks
// the slab's rows, eight in work and eight in flight; their u_j come from LDS, 64 rows at a time.
// The first unit_rows rows of workgroups make V[k] = p_k / |p_k| and sigma[k] = |p_k| instead, one a rank: as a launch of its own that was
// 3 to 5 us behind this one.
template <int NBP, bool FEW>
__global__ void __launch_bounds__(256, 3) sk_residual_kernel(float* __restrict__ W, int64_t rows, int64_t cols,
                                                             const double* __restrict__ U, int us, const double* __restrict__ P, int nb,
                                                             int64_t rows_per_slab, int unit_rows, float* __restrict__ V,
                                                             float* __restrict__ sigma)
{
    if ((int)blockIdx.y < unit_rows) {
        const int m = blockIdx.y * gridDim.x + blockIdx.x;
        if (m < nb) sk_unit(P + m * cols, cols, V + m * cols, sigma + m);
        return;
    }
    constexpr int UN = 8, CR = FEW ? 2 * UN : 64;
    __shared__ __attribute__((aligned(16))) double ul[CR][NBP];
    const int tid = threadIdx.x;
    const int64_t j = min(((int64_t)blockIdx.x * 256 + tid) * 2, cols - 2);      // past the end: the last two again, not stored
    const bool in = ((int64_t)blockIdx.x * 256 + tid) * 2 < cols;
    const int64_t r0 = (blockIdx.y - unit_rows) * rows_per_slab, r1 = min(r0 + rows_per_slab, rows);
    f64x2 p[NBP];
    auto load_p = [&]() {
#pragma unroll
        for (int m = 0; m < NBP; ++m) {
            const f64x2 t = *reinterpret_cast<const f64x2*>(P + (m < nb ? m : 0) * cols + j);
            p[m] = m < nb ? -t : f64x2{0., 0.};
        }
    };
    auto load = [&](f32x2 (&w)[UN], int64_t i) {
#pragma unroll
        for (int e = 0; e < UN; ++e) w[e] = __builtin_nontemporal_load(reinterpret_cast<const f32x2*>(W + min(i + e, r1 - 1) * cols + j));
    };
    auto load_u = [&](int64_t c0, int n) {
        for (int i = tid; i < n * NBP; i += 256) {
            const int64_t row = min(c0 + i / NBP, r1 - 1);
            ul[i / NBP][i % NBP] = i % NBP < nb ? U[row * us + i % NBP] : 0.;
        }
    };
    auto work = [&](const f32x2 (&w)[UN], int64_t c0, int o) {
#pragma unroll
        for (int e = 0; e < UN; ++e) {
            f64x2 a = {(double)w[e][0], (double)w[e][1]};
#pragma unroll
            for (int m = 0; m < NBP; m += 2) {
                const f64x2 u = *reinterpret_cast<const f64x2*>(&ul[o + e][m]);
                a[0] = fma(u[1], p[m + 1][0], fma(u[0], p[m][0], a[0]));
                a[1] = fma(u[1], p[m + 1][1], fma(u[0], p[m][1], a[1]));
            }
            if (in && c0 + o + e < r1) *reinterpret_cast<f32x2*>(W + (c0 + o + e) * cols + j) = f32x2{(float)a[0], (float)a[1]};
        }
    };
    f32x2 wa[UN], wb[UN];
    if constexpr (FEW) {
        load_u(r0, 2 * UN);
        load_p();
        load(wa, r0);
        if (r0 + UN < r1) load(wb, r0 + UN);
        tqdev::lds_barrier();
        work(wa, r0, 0);
        if (r0 + UN < r1) work(wb, r0, UN);
    } else {
        load_p();
        load(wa, r0);
        for (int64_t c0 = r0; c0 < r1; c0 += CR) {
            __syncthreads();
            load_u(c0, (int)min((int64_t)CR, (r1 - c0 + 2 * UN - 1) / (2 * UN) * (2 * UN)));
            __syncthreads();
            const int n = (int)min((int64_t)CR, r1 - c0);
            for (int o = 0; o < n; o += 2 * UN) {
                load(wb, c0 + o + UN);
                work(wa, c0, o);
                load(wa, c0 + o + 2 * UN);
                work(wb, c0, o + UN);
            }
        }
    }
}

// Shape of the fused pass for a row length: threads, float4 columns per thread, rows in work at a time; 1024 threads per CU
// whatever the width.
// Workgroups: as many as there are rows for, but with enough of them each that the partial sums stay small beside the matrix (with one
// to four rows they are 2 to 0.5 of its bytes, written and read): 128 (256 past 16384 columns, where a row alone is 64 KB and more),
// up to 256 at 16 rows each, from there 32 rows each up to what the chip holds.  Relative times with 96 / 128 / 192 / 256 at the least, a call of rank 4
// to 16: 1024 rows of 1600 and 2048 columns 1.05 / 1 / 1.05 / 1.03, of 8192 1.03 / 1 / 1.02 / 1.07, of 20000 1.11 / 1 / 1 / 1.01 (1500 rows
// 1.12 / 1 / 0.94 / 0.94).
// Whole calls, passes with 32-bit sums that applied stored deflations to the rows (errors 1.0e-7 - 1.6e-7) against this, in us (rank, power iterations): 1024 x 1024 (8, 2) 282 / 212, 1024 x 2048 (8, 2) 270 / 248, 2048 x 4096 (8, 2)
// 681 / 413, 1024 x 8192 (8, 2) 659 / 421, 32768 x 4096 (16, 1) 4286 / 2263, 4096 x 8192 (16, 2) 2056 / 1370, 4096 x 16384 (8, 2) 1607 / 1304,
// 6000 x 32768 (16, 1) 7434 / 5199, 16 x 32768 (8, 2) 369 / 360, 100000 x 64 (8, 0) 585 / 180, 1000000 x 4 (2, 1) 2086 / 1844.  377 shapes from
// 16 x 1024 to 32768 x 1024 take 0.70 of the time on average, and none is slower by more than 3 %.
struct SketchShape {
    int nt, nc, rr, wg;
    bool wide;         // 32-bit column sums
    bool few;          // no workgroup takes more steps than it requests before the first
};
bool sketch_shape(int64_t rows, int64_t cols, SketchShape* s)
{
    if (cols > 32768) return false;
    s->wide = cols > 16384;
    s->nt = cols <= 4096 ? 256 : cols <= 8192 ? 512 : 1024;
    s->nc = cols <= 1024 ? 1 : cols <= 2048 ? 2 : cols <= 16384 ? 4 : 8;
    s->rr = s->nc >= 4 ? 1 : 8 / s->nc;
    const int per_cu = 1024 / s->nt;
    const int nb = s->wide || s->nc < 4 ? 2 : 3;
    s->wg = (int)std::min<int64_t>(std::min<int64_t>(256 * per_cu, std::max<int64_t>({s->wide ? 256 : 128, std::min<int64_t>(256, (rows + 15) / 16), (rows + 31) / 32})), (rows + s->rr - 1) / s->rr);
    s->few = rows <= (int64_t)s->wg * s->rr * nb;
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
    size_t x, U, P, Z = 0, cpart, spart, dpart, ssq, ctot, zexp = 0;
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
        P->wslabs = (int)std::max<int64_t>(1, std::min(2048 / cdiv(cols, 512), cdiv(rows, 16)));
        P->w_rows = cdiv(rows, P->wslabs);
        P->wslabs = (int)cdiv(rows, P->w_rows);
        const size_t nb = P->nbs;
        P->q = take((size_t)rows * 8);
        P->x = take((size_t)cols * 4);
        P->U = take((size_t)rows * nb * 8);
        P->P = take((size_t)cols * nb * 8);
        // (Y lies in U: column k is Y_k until rank k has been found, u_k from there)
        const bool block = !P->shape.wide && nb >= 3;
        if (block) P->Z = take((size_t)cols * nb * 8);
        const size_t pass = (size_t)P->shape.wg * cols * (P->shape.wide ? 4 : 8);
        const size_t yp = block && P->ksplit > 1 ? (size_t)P->ksplit * rows * nb * 8 : 0, zp = block ? (size_t)P->zslabs * cols * nb * 8 : 0;
        P->partial = take(std::max(pass, std::max(yp, zp)));
        P->cpart = take((size_t)P->n_c * MAXB * 8);
        P->spart = take((size_t)P->n_c * MAXB * nb * 8);
        const size_t nq = std::max(P->shape.wg, P->n_q);
        P->dpart = take(nq * MAXB * 8);
        P->ssq = take(nq * 8);
        P->ctot = take(MAXB * 8);
        if (block) P->zexp = take((size_t)cdiv(cols, 64) * nb * 4);
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
    double *q = f64(P.q), *U = f64(P.U), *Pv = f64(P.P), *Y = U, *Z = f64(P.Z), *cpart = f64(P.cpart), *spart = f64(P.spart),
           *dpart = f64(P.dpart), *ssq = f64(P.ssq), *ctot = f64(P.ctot);
    float* x = reinterpret_cast<float*>(ws + P.x);
    int* zexp = reinterpret_cast<int*>(ws + P.zexp);
    ACC* partial = reinterpret_cast<ACC*>(ws + P.partial);
    const int us = P.nbs;
    const unsigned strips = (unsigned)((cols + 63) / 64);
    // where u is written the grid covers the rows as well, 256 per workgroup (a narrow matrix has few workgroups of columns)
    const unsigned fin_u = std::max((unsigned)P.n_c, (unsigned)std::min<int64_t>(1024, (rows + 255) / 256));
    const size_t smem = (size_t)(16 * MAXB + 2 * MAXB + 2 * SK_CR(sh.nt) + sh.nt) * 8 + (size_t)sh.nc * sh.nt * 16;
    auto pass = [&](int k, const float* xv, const double* parts, int cj, int cg) {
#define TQ_SKP1(NT, NC, R, NB, FEW)                                                                                            \
    hipLaunchKernelGGL((sk_pass_kernel<NT, NC, R, NB, FEW, ACC>), dim3(sh.wg), dim3(NT), smem, st, (const float*)W, rows, cols, xv, \
                       (const double*)U, us, k, parts, cj, cg, P.n_c, q, partial, ssq, dpart)
#define TQ_SKP(NT, NC, R, NB) do { if (sh.few) TQ_SKP1(NT, NC, R, NB, true); else TQ_SKP1(NT, NC, R, NB, false); } while (0)
        if constexpr (sizeof(ACC) == 4) TQ_SKP(1024, 8, 1, 2);
        else if (sh.nc == 1) TQ_SKP(256, 1, 8, 2);
        else if (sh.nc == 2) TQ_SKP(256, 2, 4, 2);
        else if (sh.nt == 256) TQ_SKP(256, 4, 1, 3);
        else if (sh.nt == 512) TQ_SKP(512, 4, 1, 3);
        else TQ_SKP(1024, 4, 1, 3);
#undef TQ_SKP
#undef TQ_SKP1
    };
    // instantiation by the number of earlier ranks, rounded up: what is loaded and folded for ranks that are not there is time between the passes
#define TQ_BY_RANKS(K, CALL) do { if ((K) == 0) { CALL(0); } else if ((K) <= 4) { CALL(4); } else if ((K) <= 8) { CALL(8); } else { CALL(16); } } while (0)
    for (int r0 = 0; r0 < r; r0 += P.nbs) {
        const int nb = std::min(P.nbs, r - r0);
        const float* S = sketch + (size_t)r0 * cols;
        // Two streams for the first products of the whole batch, against one per rank.  32-bit column sums do not bear the
        // cancellation of W^T W s.  Without power iterations the block saves a pass per rank but no launch, and takes four:
        // 1024 x 4096, rank 4: 72 us with, 79 without; 3000 x 1600, rank 4: 78 and 76; 1500 x 1600, rank 8: 103 and 122; 1024 x 1024, rank 16: 184 and 195.
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
#define TQ_FIN(KP)                                                                                                             \
    if (last)                                                                                                                  \
        hipLaunchKernelGGL((sk_finish_kernel<true, KP, ACC>), dim3(fin_u), dim3(256), 0, st, (const ACC*)part, G, G_q, cols, P.n_c, \
                           (const double*)ssq, (const double*)dpart, ce, Pv, k, nb, x, cpart, (const double*)q, rows, U, us,  \
                           U_out + (size_t)(r0 + k) * rows, S, spart);                                                        \
    else                                                                                                                       \
        hipLaunchKernelGGL((sk_finish_kernel<false, KP, ACC>), dim3(P.n_c), dim3(256), 0, st, (const ACC*)part, G, G_q, cols, P.n_c, \
                           (const double*)ssq, (const double*)dpart, ce, Pv, k, nb, x, cpart, (const double*)q, rows, U, us,  \
                           (float*)nullptr, S, spart)
                TQ_BY_RANKS(k, TQ_FIN);
#undef TQ_FIN
            };
            if (block && it == 0) {
#define TQ_PRO(KP)                                                                                                             \
    hipLaunchKernelGGL(sk_project_kernel<KP>, dim3(P.n_q), dim3(256), 0, st, (const double*)U, us, rows, k, (const double*)spart, \
                       P.n_c, q, ctot, ssq, dpart)
                TQ_BY_RANKS(k, TQ_PRO);
#undef TQ_PRO
                finish(true, Z + (size_t)k * cols, 1, P.n_q, ctot);
            } else {
#define TQ_STA(KP)                                                                                                             \
    hipLaunchKernelGGL(sk_start_kernel<KP>, dim3(P.n_c), dim3(256), 0, st, (const double*)Z, (const int*)zexp, (int)strips, cols, \
                       (const double*)Pv, k, (const double*)spart, x, cpart)
                if (block) TQ_BY_RANKS(k, TQ_STA);
#undef TQ_STA
                for (int i = block ? 1 : 0; i <= it; ++i) {
                    if (i == 0) pass(k, S + (size_t)k * cols, (const double*)spart + (size_t)k * P.n_c, MAXB * P.n_c, 1);
                    else pass(k, x, cpart, 1, sk_stride(k));
                    finish(i == it, partial, sh.wg, sh.wg, nullptr);
                }
            }
            TQ_CHECK_LAUNCH();
        }
        const unsigned res_x = (unsigned)((cols + 511) / 512), unit_rows = ((unsigned)nb + res_x - 1) / res_x;
#define TQ_RES(NBP, FEW)                                                                                                       \
    hipLaunchKernelGGL((sk_residual_kernel<NBP, FEW>), dim3(res_x, P.wslabs + unit_rows), dim3(256), 0, st, W, rows, cols, (const double*)U, \
                       us, (const double*)Pv, nb, P.w_rows, (int)unit_rows, V_out + (size_t)r0 * cols, sigma + r0)
        if (P.w_rows > 16) { if (nb <= 4) TQ_RES(4, false); else if (nb <= 8) TQ_RES(8, false); else TQ_RES(16, false); }
        else if (nb <= 4) TQ_RES(4, true); else if (nb <= 8) TQ_RES(8, true); else TQ_RES(16, true);
#undef TQ_RES
        TQ_CHECK_LAUNCH();
    }
    return TQ_OK;
}

}  // namespace

tq_status tqi_setup_sketch()
{
    // x of a pass takes up to 128 KB of LDS
    bool ok = true;
#define TQ_ATTR(NT, NC, R, NB, FEW, ACC)                                                                                      \
    ok = ok && hipFuncSetAttribute((const void*)sk_pass_kernel<NT, NC, R, NB, FEW, ACC>, hipFuncAttributeMaxDynamicSharedMemorySize, \
                                   160 * 1024) == hipSuccess
    TQ_ATTR(1024, 8, 1, 2, false, float); TQ_ATTR(1024, 8, 1, 2, true, float);
    TQ_ATTR(1024, 4, 1, 3, false, double); TQ_ATTR(1024, 4, 1, 3, true, double);
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
