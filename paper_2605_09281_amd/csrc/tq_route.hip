// tq_route (top-k selection and routing weights) and the token -> expert permutation with
// prefix-sum offsets (histogram, scan, stable scatter) that tq_permute exports and tq_moe_forward
// runs as its first step.
#include "tq_prep.h"

namespace {

constexpr int kMaxPerLane = 16;  // E <= 64 * 16

// One wavefront per token.  Lane l holds the scores of experts l, l+64, l+128, ... (PL of them: the per-lane scans
// are unrolled to the number of experts a lane can hold, not to the maximum).
// Each of the k rounds takes the wave-wide maximum under the order (score desc, index asc).
// One selection round over the scores a wave holds (lane l: experts l, l + 64, ...; `taken` marks the ones already
// chosen or past E): the wave-wide maximum under the order (score desc, index asc), marked as taken in its lane.
template <int PL>
__device__ inline void wave_select_round(const float (&v)[PL], uint32_t& taken, int lane, float& bv, int& be)
{
    // best candidate of this lane: ascending index scan with a strict compare keeps the lowest index
    bv = 0.f;
    be = 0x7FFFFFFF;
#pragma unroll
    for (int i = 0; i < PL; ++i) {
        if (!((taken >> i) & 1u)) {
            if (be == 0x7FFFFFFF || v[i] > bv) { bv = v[i]; be = lane + 64 * i; }
        }
    }
    // wave-wide arg-max under (score desc, index asc); lanes with nothing left carry index INT_MAX
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        float ov = __shfl_xor(bv, off);
        int oe = __shfl_xor(be, off);
        bool take = (oe != 0x7FFFFFFF) && (be == 0x7FFFFFFF || ov > bv || (ov == bv && oe < be));
        if (take) { bv = ov; be = oe; }
    }
    if ((be & 63) == lane) taken |= 1u << (be >> 6);
}

template <int PL>
__device__ inline void wave_load_scores(const float* __restrict__ logits_row, const float* __restrict__ bias, int E, int lane,
                                        float (&v)[PL], uint32_t& taken)
{
    taken = 0;
#pragma unroll
    for (int i = 0; i < PL; ++i) {
        int e = lane + 64 * i;
        float s = -INFINITY;
        if (e < E) {
            s = logits_row[e];
            if (bias) s = s + bias[e];
        } else {
            taken |= 1u << i;
        }
        v[i] = s;
    }
}

template <int PL>
__global__ void __launch_bounds__(256) route_kernel(const float* __restrict__ logits,
                                                    const float* __restrict__ bias, int T, int E, int k,
                                                    int32_t* __restrict__ topk_idx, float* __restrict__ topk_w)
{
    const int lane = threadIdx.x & 63;
    const int t = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    if (t >= T) return;
    float v[PL];
    uint32_t taken;
    wave_load_scores<PL>(logits + (size_t)t * E, bias, E, lane, v, taken);
    float first = 0.f, denom = 0.f, my_p = 0.f;
    for (int j = 0; j < k; ++j) {
        float bv;
        int be;
        wave_select_round<PL>(v, taken, lane, bv, be);
        if (j == 0) first = bv;
        float p = expf(bv - first);       // the same value in every lane
        denom += p;
        if (lane == j) my_p = p;          // lane j keeps the unnormalised weight of slot j (k <= 64)
        if (lane == 0) topk_idx[(size_t)t * k + j] = be;
    }
    if (lane < k) topk_w[(size_t)t * k + lane] = my_p / denom;
}

// Layers of at most 256 experts and 16 selections: a row of 16 lanes per token, lane l of it holding experts l, l + 16,
// ... (PL of them), so that a wave routes four tokens and every step of the arg-max stays inside a row, where lanes
// exchange values by DPP.  With a wave per token (route_kernel) each round is twelve exchanges through the LDS crossbar,
// which is what that kernel is bound by: 8192 tokens of 128 experts, top-8, 15.4 us there and 5.6 us here (4 MB of scores: the rest is latency of the rounds).
// A score is held as an integer that orders the same way, so a round is a maximum, then the lowest expert that has it:
// the order of route_kernel (score desc, index asc; -0 counts as +0), and its arithmetic on the scores.  An expert already
// chosen (or past E) orders below everything.  NaN scores are not supported by the entry points: here they order below every number, in
// the other two forms by where they stand.
constexpr int32_t ROUTE_TAKEN = (int32_t)0x80000000, ROUTE_NAN = ROUTE_TAKEN + 1;
__device__ inline int32_t route_key(float s)
{
    const int32_t b = __float_as_int(s + 0.0f);          // -0 + 0 = +0
    const int32_t key = b < 0 ? b ^ 0x7FFFFFFF : b;
    return s != s ? ROUTE_NAN : key;
}
__device__ inline float route_score(int32_t key) { return __int_as_float(key < 0 ? key ^ 0x7FFFFFFF : key); }

template <int CTRL>
__device__ inline int row_dpp(int v) { return __builtin_amdgcn_update_dpp(v, v, CTRL, 0xF, 0xF, false); }
__device__ inline int row_max(int v)          // rotations by 8, 4, 2, 1: every lane of the row ends with the maximum
{
    v = max(v, row_dpp<0x128>(v));
    v = max(v, row_dpp<0x124>(v));
    v = max(v, row_dpp<0x122>(v));
    return max(v, row_dpp<0x121>(v));
}
__device__ inline int row_min(int v)
{
    v = min(v, row_dpp<0x128>(v));
    v = min(v, row_dpp<0x124>(v));
    v = min(v, row_dpp<0x122>(v));
    return min(v, row_dpp<0x121>(v));
}

template <int PL>
__global__ void __launch_bounds__(256) route_row_kernel(const float* __restrict__ logits, const float* __restrict__ bias,
                                                        int T, int E, int k, int32_t* __restrict__ topk_idx,
                                                        float* __restrict__ topk_w)
{
    const int sub = threadIdx.x & 15;
    const int t_raw = blockIdx.x * 16 + (threadIdx.x >> 4);
    const int t = min(t_raw, T - 1);          // a row past the end repeats the last token and stores nothing
    const float* row = logits + (size_t)t * E;
    float v[PL], b[PL];
#pragma unroll
    for (int i = 0; i < PL; ++i) {            // all loads are issued together, from addresses that exist
        const int e = min(sub + 16 * i, E - 1);
        v[i] = row[e];
        b[i] = bias ? bias[e] : 0.f;
    }
    int32_t key[PL];
#pragma unroll
    for (int i = 0; i < PL; ++i) {
        const float s = bias ? v[i] + b[i] : v[i];
        key[i] = sub + 16 * i < E ? route_key(s) : ROUTE_TAKEN;
    }
    float first = 0.f, denom = 0.f, my_p = 0.f;
    int my_e = 0;
    for (int j = 0; j < k; ++j) {             // k <= E: there is an expert left in every round
        int m = key[0];
#pragma unroll
        for (int i = 1; i < PL; ++i) m = max(m, key[i]);
        m = row_max(m);
        int be = 0x7FFFFFFF;
#pragma unroll
        for (int i = PL - 1; i >= 0; --i) be = key[i] == m ? sub + 16 * i : be;
        be = row_min(be);
#pragma unroll
        for (int i = 0; i < PL; ++i) key[i] = be == sub + 16 * i ? ROUTE_TAKEN : key[i];
        const float bv = route_score(m);
        if (j == 0) first = bv;
        const float p = expf(bv - first);     // the same value in every lane of the row
        denom += p;
        if (sub == j) { my_p = p; my_e = be; }
    }
    if (t_raw < T && sub < k) {
        topk_idx[(size_t)t * k + sub] = my_e;
        topk_w[(size_t)t * k + sub] = my_p / denom;
    }
}

// The routing of a decode batch inside the permutation's launch (at most 64 tokens and 16 experts): one LANE per
// token scans its scores serially, the same order (score desc, index asc) and the same arithmetic as route_kernel,
// so the results are identical bit for bit.  Bound by one wave's instructions: a lane holds its token's scores in registers.  Staged through
// LDS they cost 32 divisions by E and a dependent read per score and round (whole calls: 16 experts of 512 x 1024, top-2, 64 tokens
// 33.7 -> 31.6 us; of 1024 x 1024, top-8, 32 tokens 62.8 -> 59.1; 12 of 512 x 1024, top-6, 32 tokens 38.0 -> 36.1; 8 of 4096 x 14336, 1 token
// 60.4 -> 60.0).  The results land in LDS (ridx, rw: [T * k]) for the permutation that follows and in memory for the caller.
__device__ inline void route_small(const TqRouteIn& R, int T, int E, int k, int32_t* ridx, float* rw, int lane)
{
    constexpr int NE = 16;
    float s[NE];
    const float* row = R.logits + (size_t)min(lane, T - 1) * E;
#pragma unroll
    for (int e = 0; e < NE; ++e) s[e] = row[min(e, E - 1)];
    if (R.bias) {
#pragma unroll
        for (int e = 0; e < NE; ++e) s[e] = s[e] + R.bias[min(e, E - 1)];
    }
    if (lane < T) {
        uint32_t taken = ~0u << E;
        float first = 0.f, denom = 0.f;
        for (int j = 0; j < k; ++j) {
            float bv = 0.f;
            int be = -1;
#pragma unroll
            for (int e = 0; e < NE; ++e)
                if (!((taken >> e) & 1u) && (be < 0 || s[e] > bv)) { bv = s[e]; be = e; }
            taken |= 1u << be;
            if (j == 0) first = bv;
            const float p = expf(bv - first);
            denom += p;
            ridx[lane * k + j] = be;
            rw[lane * k + j] = p;
        }
        for (int j = 0; j < k; ++j) rw[lane * k + j] = rw[lane * k + j] / denom;
    }
    __syncthreads();
    for (int a = lane; a < T * k; a += 64) {
        R.idx_out[a] = ridx[a];
        R.w_out[a] = rw[a];
    }
}

// The expert of assignment (t, j) recomputed by one wave from the token's scores (E <= 64): the workgroups that share
// the permutation's launch cannot wait for its routing results.
__device__ inline int route_expert_of(const TqRouteIn& R, int t, int j, int E, int lane)
{
    float v[1];
    uint32_t taken;
    wave_load_scores<1>(R.logits + (size_t)t * E, R.bias, E, lane, v, taken);
    int be = 0;
    for (int q = 0; q <= j; ++q) {
        float bv;
        wave_select_round<1>(v, taken, lane, bv, be);
    }
    return be;
}

// ---------------------------------------------------------------------------------------------
// Permutation.
//   permute_small_kernel: the whole of it in one wavefront, up to TQ_PERM_CHUNK assignments (decode batches)
//   permute_place_kernel: larger batches, a workgroup per TQ_PLACE_CHUNK assignments; past TQ_PLACE_COUNT_SELF of them
//                         after a launch of permute_hist_kernel (and of permute_scan_kernel where there are many counts)
//
// Row-tile tables: for each tiling (32, 128, 16, 64 rows) the list of (expert, first slot) of every tile,
// expert-major; their lengths go to ctrl[1], ctrl[2], ctrl[4], ctrl[5]; ctrl[3] = number of rows in total.
__device__ inline int tile_rows_of(int which) { return which == 0 ? 32 : which == 1 ? 128 : which == 2 ? 16 : 64; }
__device__ inline int tile_ctrl_of(int which) { return which == 0 ? 1 : which == 1 ? 2 : which == 2 ? 4 : 5; }

__device__ inline int wave_incl_scan(int v, int lane)
{
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        int o = __shfl_up(v, off);
        if (lane >= off) v += o;
    }
    return v;
}

// One wavefront: out[0..n] = exclusive prefix sum of f(in[i]); returns the total.  in/out live in LDS.
template <typename F>
__device__ inline int wave_excl_scan(const int32_t* in, int32_t* out, int n, int lane, F f)
{
    int carry = 0;
    for (int i0 = 0; i0 < n; i0 += 64) {
        int i = i0 + lane;
        int v = i < n ? f(in[i]) : 0;
        int inc = wave_incl_scan(v, lane);
        if (i < n) out[i] = carry + inc - v;
        carry += __shfl(inc, 63);
    }
    if (lane == 0) out[n] = carry;
    return carry;
}

__device__ inline bool blob_header_ok(const TqBlobHeader* hdr, const TqBlobHeader& expect)
{
    return hdr->magic == expect.magic && hdr->version == expect.version && hdr->n_experts == expect.n_experts &&
           hdr->n_shared == expect.n_shared && hdr->hidden == expect.hidden && hdr->ffn == expect.ffn &&
           hdr->group == expect.group && hdr->bits == expect.bits && hdr->rank == expect.rank &&
           hdr->code_words == expect.code_words && hdr->factor_fp8 == expect.factor_fp8 && hdr->tiles_m == expect.tiles_m && hdr->tiles_n == expect.tiles_n &&
           hdr->expert_stride == expect.expert_stride;
}

constexpr int TQ_PLACE_THREADS = 512, TQ_PLACE_WAVES = TQ_PLACE_THREADS / 64;
constexpr int TQ_PLACE_CHUNK = 1024;                                   // assignments of one workgroup
constexpr int TQ_PLACE_ROUNDS = TQ_PLACE_CHUNK / TQ_PLACE_THREADS;     // 64-wide rounds of one wave
// Up to this many assignments every workgroup of permute_place_kernel counts all of them itself (at most eight loads
// per thread, one launch); beyond, permute_hist_kernel counts each chunk once and the workgroups add up the counts.
// Measured, one launch against two: 2048 assignments of 8 / 128 experts 5.5 / 6.0 us against 7.4 / 7.9, 4096 6.1 / 6.3 against
// 7.5 / 8.0; with 32 loads per thread 8192 take 8.3 / 7.9 against 7.6 / 8.4, 16384 10.9 / 8.9 against 7.6 / 9.0.
constexpr int TQ_PLACE_COUNT_SELF = 4096;
// From this many counts (chunks x experts) permute_scan_kernel adds them up; below, every workgroup of permute_place_kernel
// adds up all of them, which saves that launch but reads (chunks)^2 x experts words in all.  Measured, without the launch against with it:
// at 32768 counts 17.2 us against 16.9 (1024 experts), 12.8 / 12.8 (128), 14.0 / 14.3 (64), 63 / 44 (8); at a quarter of them
// 14.1 / 16.2, 9.2 / 11.9, 8.9 / 12.4, 14.9 / 17.0; at four times 28.8 / 18.6, 48 / 23, 279 / 56 (8 times, 64 experts); 4 M assignments of
// 1024 experts 4495 / 119.
constexpr int64_t TQ_PLACE_SCAN_WORDS = 32768;

// hist[b][e] = assignments of expert e in chunk b; hist[gridDim.x * E + b] = whether the chunk holds an invalid index
__global__ void __launch_bounds__(TQ_PLACE_THREADS) permute_hist_kernel(const int32_t* __restrict__ idx, int64_t n_assign,
                                                                        int E, int32_t* __restrict__ hist)
{
    extern __shared__ int32_t cnt[];       // [E] | flag
    const int tid = threadIdx.x, b = blockIdx.x;
    int ev[TQ_PLACE_ROUNDS];
#pragma unroll
    for (int r = 0; r < TQ_PLACE_ROUNDS; ++r) {
        const int64_t a = (int64_t)b * TQ_PLACE_CHUNK + r * TQ_PLACE_THREADS + tid;
        ev[r] = a < n_assign ? idx[a] : E;
    }
    for (int e = tid; e <= E; e += TQ_PLACE_THREADS) cnt[e] = 0;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < TQ_PLACE_ROUNDS; ++r) {
        const int64_t a = (int64_t)b * TQ_PLACE_CHUNK + r * TQ_PLACE_THREADS + tid;
        if (ev[r] >= 0 && ev[r] < E) atomicAdd(&cnt[ev[r]], 1);
        else if (a < n_assign) atomicOr(&cnt[E], 1);
    }
    __syncthreads();
    for (int e = tid; e < E; e += TQ_PLACE_THREADS) hist[(size_t)b * E + e] = cnt[e];
    if (tid == 0) hist[(size_t)gridDim.x * E + b] = cnt[E];
}

// From TQ_PLACE_SCAN_WORDS counts on: hist[b][e] becomes the number of assignments of expert e in the chunks before b, and
// hist[nb * E + nb + e] their total, so that a workgroup of permute_place_kernel reads 2 E words instead of all nb * E.
// A thread owns one expert (of `ep` per workgroup, ep a power of two up to 32: whole lines of a row) and one of 1024 / ep runs of
// consecutive chunks: it sums its run, the runs are scanned in LDS, and it rewrites its run.
constexpr int TQ_SCAN_THREADS = 1024;
__global__ void __launch_bounds__(TQ_SCAN_THREADS) permute_scan_kernel(int32_t* __restrict__ hist, int nb, int E, int ep)
{
    __shared__ int32_t sums[TQ_SCAN_THREADS];
    const int tid = threadIdx.x, run = tid / ep, runs = TQ_SCAN_THREADS / ep;
    const int e = blockIdx.x * ep + (tid & (ep - 1));
    const int per = (nb + runs - 1) / runs;
    const int64_t c0 = (int64_t)run * per;
    const int n = e < E && c0 < nb ? (int)min((int64_t)per, nb - c0) : 0;
    int32_t* h = hist + c0 * E + e;
    int tot = 0;
#pragma unroll 8
    for (int i = 0; i < n; ++i) tot += h[(size_t)i * E];
    sums[tid] = tot;
    __syncthreads();
    for (int off = ep; off < TQ_SCAN_THREADS; off *= 2) {
        const int o = tid >= off ? sums[tid - off] : 0;
        __syncthreads();
        sums[tid] += o;
        __syncthreads();
    }
    int before = sums[tid] - tot;
    int i = 0;
    for (; i + 8 <= n; i += 8) {
        int v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = h[(size_t)(i + u) * E];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            h[(size_t)(i + u) * E] = before;
            before += v[u];
        }
    }
    for (; i < n; ++i) {
        const int v = h[(size_t)i * E];
        h[(size_t)i * E] = before;
        before += v;
    }
    if (run == runs - 1 && e < E) hist[(size_t)nb * E + nb + e] = sums[tid];
}

// orders one wavefront's LDS reads before its later writes (and the writes before the next reads) where its workgroup's
// other waves do not take part
__device__ inline void wave_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// writes the row-tile tables from offs[0..ne] (LDS); `sm_base` is LDS scratch of TQ_N_TILINGS*(ne+1) ints;
// tile_row0 holds 2 * TQ_N_TILINGS * rt_max ints: the first slots, then the row counts.  Workgroup `part` of `nparts`
// (each with all of offs) writes its share of the entries; the first one writes the counts.
__device__ inline void build_tile_tables(const int32_t* offs, int32_t* sm_base, int ne, int32_t* tile_e,
                                         int32_t* tile_row0, int rt_max, int32_t* ctrl, int tid, int nthreads,
                                         int tilings, int part = 0, int nparts = 1)
{
    // per tiling: tiles of expert e = ceil(count/bm); scan by wavefront `which` (or by wave 0 in turn)
    const int lane = tid & 63, wave = tid >> 6, nwaves = nthreads >> 6;
    for (int which = wave; which < TQ_N_TILINGS; which += nwaves) {
        if (!((tilings >> which) & 1)) continue;       // tilings no kernel of this forward reads (their counts stay 0)
        const int bm = tile_rows_of(which);
        int32_t* base = sm_base + which * (ne + 1);
        int carry = 0;
        for (int i0 = 0; i0 < ne; i0 += 64) {
            int i = i0 + lane;
            int v = i < ne ? (offs[i + 1] - offs[i] + bm - 1) / bm : 0;
            int inc = wave_incl_scan(v, lane);
            if (i < ne) base[i] = carry + inc - v;
            carry += __shfl(inc, 63);
        }
        if (lane == 0) {
            base[ne] = carry;
            if (part == 0) ctrl[tile_ctrl_of(which)] = carry < rt_max ? carry : rt_max;
        }
    }
    __syncthreads();
    // one entry per thread: the expert of tile n is found by bisection over the per-expert first tiles
    for (int which = 0; which < TQ_N_TILINGS; ++which) {
        if (!((tilings >> which) & 1)) continue;
        const int bm = tile_rows_of(which);
        const int32_t* base = sm_base + which * (ne + 1);
        const int total = base[ne] < rt_max ? base[ne] : rt_max;
        int32_t* te = tile_e + (size_t)which * rt_max;
        int32_t* tr = tile_row0 + (size_t)which * rt_max;
        for (int n = part * nthreads + tid; n < total; n += nparts * nthreads) {
            int lo = 0, hi = ne - 1;          // largest e with base[e] <= n (experts without rows share a base)
            while (lo < hi) {
                int mid = (lo + hi + 1) >> 1;
                if (base[mid] <= n) lo = mid; else hi = mid - 1;
            }
            te[n] = lo;
            tr[n] = offs[lo] + (n - base[lo]) * bm;
            // the tile's row count, behind the first-slot tables: saves the decode kernels a dependent load of offsets
            tr[n + (size_t)TQ_N_TILINGS * rt_max] = min(bm, offs[lo + 1] - tr[n]);
        }
    }
}

// Batches past one chunk: a workgroup places TQ_PLACE_CHUNK assignments, its eight waves 128 each.  It takes the number
// of assignments of every expert in all chunks and in the chunks before its own (from `hist`, with `scanned` added up there
// already, or by counting them when hist is null), scans the totals into the offsets, turns its waves' own counts into
// cursors and places 64 assignments per round, ranked by ballots: chunk-major, stable inside a chunk.  The work of every workgroup is the same few steps,
// so nothing waits on one workgroup's scan: the five launches of one wave or one workgroup each that did this before
// (clear, histogram, chunk scan, scan with tables, scatter) were latency: 9186 assignments of 64 experts 35 us in five launches,
// 14 us in two here; 4096 assignments of 60 experts 17 us in one workgroup of 16 waves, 9.6 us here.
// With PREP the workgroups past the first nb derive what the tiled kernels read beside the blob (tq_prep.h).
struct NoPrep {};
template <bool PREP>
__global__ void __launch_bounds__(TQ_PLACE_THREADS) permute_place_kernel(
    const int32_t* __restrict__ idx, const float* __restrict__ w, int64_t n_assign, int E, int S, int T, int k,
    const int32_t* __restrict__ hist, int scanned, int32_t* __restrict__ offsets, int32_t* __restrict__ slot_of, int slot_stride,
    int32_t* __restrict__ src_of, int32_t* __restrict__ row_token, float* __restrict__ row_w, int32_t* __restrict__ tile_e,
    int32_t* __restrict__ tile_row0, int rt_max, int32_t* __restrict__ ctrl, int32_t* __restrict__ err_flag,
    const TqBlobHeader* __restrict__ hdr, TqBlobHeader expect, int check_blob, int32_t* __restrict__ zero_buf, int zero_n,
    int tilings, int nb, std::conditional_t<PREP, TqPrep, NoPrep> P)
{
    if constexpr (PREP) {
        if ((int)blockIdx.x >= nb) {
            tq_prep_wave(P, (blockIdx.x - nb) * (TQ_PLACE_THREADS / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), threadIdx.x & 63);
            return;
        }
    }
    extern __shared__ int32_t sm[];   // before[E] | totals[ne] | offs[ne+1] | tile scratch TQ_N_TILINGS*(ne+1) | cursor[waves][E] | flags
    const int ne = E + S;
    int32_t* before = sm;
    int32_t* totals = before + E;
    int32_t* offs = totals + ne;
    int32_t* tsm = offs + ne + 1;
    int32_t* cursor = tsm + TQ_N_TILINGS * (ne + 1);
    int32_t* flagw = cursor + TQ_PLACE_WAVES * E;
    constexpr int NT = TQ_PLACE_THREADS;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int b = blockIdx.x;
    const int64_t a_wave = (int64_t)b * TQ_PLACE_CHUNK + wave * (64 * TQ_PLACE_ROUNDS);

    int ev[TQ_PLACE_ROUNDS];          // expert of this lane's assignment in each round; -1: invalid or past the end
    float wv[TQ_PLACE_ROUNDS];
#pragma unroll
    for (int r = 0; r < TQ_PLACE_ROUNDS; ++r) {
        const int64_t a = a_wave + r * 64 + lane;
        ev[r] = a < n_assign ? idx[a] : -1;
        wv[r] = (w && a < n_assign) ? w[a] : 1.0f;
        if (ev[r] >= E) ev[r] = -1;
    }
    TqBlobHeader hv = expect;
    if (check_blob && b == 0 && tid == 0) hv = *hdr;
    if (b == 0 && ctrl && tid < 64) ctrl[tid] = 0;
    for (int i = b * NT + tid; i < zero_n; i += nb * NT) zero_buf[i] = 0;
    for (int i = tid; i < E; i += NT) before[i] = 0;
    for (int i = tid; i < ne; i += NT) totals[i] = i < E ? 0 : T;
    for (int i = tid; i < TQ_PLACE_WAVES * E; i += NT) cursor[i] = 0;
    if (tid == 0) *flagw = 0;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < TQ_PLACE_ROUNDS; ++r)
        if (ev[r] >= 0) atomicAdd(&cursor[wave * E + ev[r]], 1);
    if (hist && scanned) {
        for (int e = tid; e < E; e += NT) {
            totals[e] = hist[(size_t)nb * E + nb + e];
            before[e] = hist[(size_t)b * E + e];
        }
    } else if (hist) {
        // threads side by side on the experts, the chunks dealt to NT / ep groups of them
        int ep = 1;
        while (ep < E && ep < NT) ep *= 2;
        const int np = NT / ep;
        for (int e = tid & (ep - 1); e < E; e += ep) {
            int tot = 0, bef = 0;
#pragma unroll 8
            for (int c = tid / ep; c < nb; c += np) {
                const int v = hist[(size_t)c * E + e];
                tot += v;
                bef += c < b ? v : 0;
            }
            atomicAdd(&totals[e], tot);
            atomicAdd(&before[e], bef);
        }
    } else {
        constexpr int NL = TQ_PLACE_COUNT_SELF / NT;
        int av[NL];
#pragma unroll
        for (int u = 0; u < NL; ++u) av[u] = idx[min((int64_t)u * NT + tid, n_assign - 1)];
#pragma unroll
        for (int u = 0; u < NL; ++u) {
            const int64_t a = (int64_t)u * NT + tid;
            if (a < n_assign) {
                if (av[u] >= 0 && av[u] < E) {
                    atomicAdd(&totals[av[u]], 1);
                    if (a < (int64_t)b * TQ_PLACE_CHUNK) atomicAdd(&before[av[u]], 1);
                } else {
                    atomicOr(flagw, TQ_FLAG_BIT_RANGE);
                }
            }
        }
    }
    if (hist && b == 0) {
        int bad = 0;
#pragma unroll 8
        for (int c = tid; c < nb; c += NT) bad |= hist[(size_t)nb * E + c];
        if (bad) atomicOr(flagw, TQ_FLAG_BIT_RANGE);
    }
    if (check_blob && b == 0 && tid == 0 && !blob_header_ok(&hv, expect)) atomicOr(flagw, TQ_FLAG_BIT_BLOB);
    __syncthreads();
    if (wave == 0) {
        const int total = wave_excl_scan(totals, offs, ne, lane, [](int v) { return v; });
        if (b == 0 && lane == 0 && ctrl) ctrl[3] = total;
    }
    __syncthreads();
    if (b == 0)
        for (int e = tid; e <= ne; e += NT) offsets[e] = offs[e];
    for (int e = tid; e < E; e += NT) {      // the waves' counts become their cursors
        int run = offs[e] + before[e];
#pragma unroll
        for (int v = 0; v < TQ_PLACE_WAVES; ++v) {
            const int c = cursor[v * E + e];
            cursor[v * E + e] = run;
            run += c;
        }
    }
    if (tile_e) build_tile_tables(offs, tsm, ne, tile_e, tile_row0, rt_max, ctrl, tid, NT, tilings, b, nb);
    __syncthreads();
    int32_t* cur = cursor + wave * E;
#pragma unroll
    for (int r = 0; r < TQ_PLACE_ROUNDS; ++r) {
        const int64_t a = a_wave + r * 64 + lane;
        const int e = ev[r];
        // lanes holding the same expert: intersect, bit by bit of e, the ballots that agree with this lane
        uint64_t same = __ballot(e >= 0);
        for (int bit = 0; (1 << bit) < E; ++bit) {
            const uint64_t bal = __ballot((e >> bit) & 1);
            same &= ((e >> bit) & 1) ? bal : ~bal;
        }
        const int rank = __popcll(same & ((1ull << lane) - 1ull));
        const bool last = (same >> lane) <= 1ull;      // no higher lane with this expert
        const int slot = e >= 0 ? cur[e] + rank : -1;
        wave_fence();
        if (e >= 0 && last) cur[e] = slot + 1;         // the last lane of each expert moves its cursor
        wave_fence();
        if (a < n_assign) {
            const int t = (int)(a / k), j = (int)(a % k);
            if (slot_of) slot_of[(size_t)t * slot_stride + j] = slot;
            if (slot >= 0) {
                if (src_of) src_of[slot] = (int32_t)a;
                if (row_token) row_token[slot] = t;
                if (row_w) row_w[slot] = wv[r];
            }
        }
    }
    // shared experts: every token, weight 1, identity order
    const int64_t n_sh = (int64_t)S * T;
    for (int64_t i = (int64_t)b * NT + tid; i < n_sh; i += (int64_t)nb * NT) {
        const int s = (int)(i / T), t = (int)(i % T);
        const int slot = offs[E + s] + t;
        if (slot_of) slot_of[(size_t)t * slot_stride + k + s] = slot;
        if (src_of) src_of[slot] = (int32_t)(n_assign + i);
        if (row_token) row_token[slot] = t;
        if (row_w) row_w[slot] = 1.0f;
    }
    if (b == 0 && tid == 0) {
        const int flags = *flagw;
        if (flags && err_flag) atomicOr(err_flag, flags);
        // a blob that does not belong to the descriptor: no row tiles and no rows, so that every later kernel of the
        // forward ends at once instead of indexing the blob with the wrong geometry
        if ((flags & TQ_FLAG_BIT_BLOB) && ctrl) { ctrl[1] = 0; ctrl[2] = 0; ctrl[3] = 0; ctrl[4] = 0; ctrl[5] = 0; }
    }
}

__device__ inline void permute_small_body(const int32_t* __restrict__ idx, const float* __restrict__ w,
                                                           int n_assign, int E, int S, int T, int k,
                                                           int32_t* __restrict__ offsets, int32_t* __restrict__ slot_of,
                                                           int slot_stride, int32_t* __restrict__ src_of,
                                                           int32_t* __restrict__ row_token, float* __restrict__ row_w,
                                                           int32_t* __restrict__ tile_e, int32_t* __restrict__ tile_row0,
                                                           int rt_max, int32_t* __restrict__ ctrl,
                                                           int32_t* __restrict__ err_flag,
                                                           const TqBlobHeader* __restrict__ hdr, TqBlobHeader expect,
                                                           int check_blob, int32_t* __restrict__ zero_buf, int zero_n,
                                                           int tilings)
{
    extern __shared__ int32_t sm[];   // counts[ne] | offs[ne+1] | cursor[E] | tile scratch TQ_N_TILINGS*(ne+1)
    const int ne = E + S, lane = threadIdx.x;
    int32_t* counts = sm;
    int32_t* offs = counts + ne;
    int32_t* cursor = offs + ne + 1;
    int32_t* tsm = cursor + E;
    // everything this wave reads from memory is requested first (one round trip instead of three): the
    // assignments and weights of up to four rounds of 64, and the blob header
    constexpr int NR = TQ_PERM_CHUNK / 64;
    int ev[NR];
    float wv[NR];
#pragma unroll
    for (int j = 0; j < NR; ++j) {
        ev[j] = -2;                                  // past the end: neither counted nor flagged
        wv[j] = 1.0f;
    }
    if (n_assign > 0) {                              // an empty batch has no first element to clamp to
#pragma unroll
        for (int j = 0; j < NR; ++j) {
            const int a = j * 64 + lane;
            const int ac = min(a, n_assign - 1);
            const int ej = idx[ac];
            const float wj = w ? w[ac] : 1.0f;
            if (a < n_assign) { ev[j] = ej; wv[j] = wj; }
        }
    }
    TqBlobHeader hv = expect;
    if (check_blob) hv = *hdr;
    if (ctrl) ctrl[lane] = 0;
    for (int i = lane; i < zero_n; i += 64) zero_buf[i] = 0;
    for (int e = lane; e < ne; e += 64) counts[e] = e < E ? 0 : T;
    __syncthreads();
    bool bad = false;
#pragma unroll
    for (int j = 0; j < NR; ++j) {
        if (ev[j] >= 0 && ev[j] < E) atomicAdd(&counts[ev[j]], 1);
        else if (ev[j] != -2) { bad = true; ev[j] = -1; }
    }
    __syncthreads();
    int flags = __ballot(bad) ? TQ_FLAG_BIT_RANGE : 0;
    if (check_blob && !blob_header_ok(&hv, expect)) flags |= TQ_FLAG_BIT_BLOB;
    int total = wave_excl_scan(counts, offs, ne, lane, [](int v) { return v; });
    __syncthreads();
    for (int e = lane; e <= ne; e += 64) offsets[e] = offs[e];
    for (int e = lane; e < E; e += 64) cursor[e] = offs[e];
    __syncthreads();
    if (ctrl && lane == 0) ctrl[3] = total;
    if (tile_e) build_tile_tables(offs, tsm, ne, tile_e, tile_row0, rt_max, ctrl, lane, 64, tilings);
    __syncthreads();
    // stable placement, 64 assignments per round in order (same ranking as permute_place_kernel)
#pragma unroll
    for (int j = 0; j < NR; ++j) {
        if (j * 64 >= n_assign) break;
        const int a = j * 64 + lane;
        const int e = ev[j] >= 0 ? ev[j] : -1;
        uint64_t same = __ballot(e >= 0);
        for (int bit = 0; (1 << bit) < E; ++bit) {
            const uint64_t bal = __ballot((e >> bit) & 1);
            same &= ((e >> bit) & 1) ? bal : ~bal;
        }
        const int before = __popcll(same & ((1ull << lane) - 1ull));
        const bool last = (same >> lane) <= 1ull;
        const int slot = e >= 0 ? cursor[e] + before : -1;
        __syncthreads();
        if (e >= 0 && last) cursor[e] = slot + 1;
        __syncthreads();
        if (a < n_assign) {
            const int t = a / k, jj = a % k;
            if (slot_of) slot_of[(size_t)t * slot_stride + jj] = slot;
            if (slot >= 0) {
                if (src_of) src_of[slot] = (int32_t)a;
                if (row_token) row_token[slot] = t;
                if (row_w) row_w[slot] = wv[j];
            }
        }
    }
    for (int i = lane; i < S * T; i += 64) {
        int s = i / T, t = i % T;
        int slot = offs[E + s] + t;
        if (slot_of) slot_of[(size_t)t * slot_stride + k + s] = slot;
        if (src_of) src_of[slot] = n_assign + i;
        if (row_token) row_token[slot] = t;
        if (row_w) row_w[slot] = 1.0f;
    }
    if (flags && lane == 0 && err_flag) atomicOr(err_flag, flags);
    // a blob that does not belong to the descriptor must not be indexed with the descriptor's geometry: with no
    // row tiles and no rows every later kernel of the forward ends at once
    if ((flags & TQ_FLAG_BIT_BLOB) && ctrl && lane == 0) { ctrl[1] = 0; ctrl[2] = 0; ctrl[3] = 0; ctrl[4] = 0; ctrl[5] = 0; }
}

// One workgroup per (assignment v, part, 32-column tile of t), a wave per 256-wide slice of the contraction: see TqPreByAssign.  Plain fp32 FMAs on
// the exact values of x (bf16) and A (fp16, or fp8 with FP8), the two halves of a 16-wide step in the two halves of a wave; the slices are
// added in order through LDS.
template <bool FP8>
__device__ inline void pre_by_assign_block(const TqPreByAssign& P, const int32_t* __restrict__ idx, int T, int E, int k,
                                           int b, const TqRouteIn* route = nullptr)
{
    __shared__ float red[TQ_PRE_PART_SLICES][32];
    __shared__ __attribute__((aligned(16))) uint2 xl[TQ_PRE_PART_SLICES][64];      // each wave's slice of the row
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int ta = b % P.na_tiles, part = b / P.na_tiles % P.n_parts;
    const int v = b / (P.na_tiles * P.n_parts), slice = part * TQ_PRE_PART_SLICES + w;
    if (v >= P.a_tot) return;
    int e, t;
    if (v < T * k) {
        t = v / k;
        e = route ? route_expert_of(*route, t, v % k, E, lane) : idx[v];
        if (e < 0 || e >= E) return;      // dropped assignments have no row
    }
    else { const int q = v - T * k; e = E + q / T; t = q % T; }
    const int col = lane & 31, hf = lane >> 5;
    const int ksteps = P.H / 16;
    const uint16_t* xrow = P.x + (size_t)t * P.H;
    const uint4* af = reinterpret_cast<const uint4*>(tq_afrag_base(P.blob, P.expert_stride, P.sec, P.fm, 0, e));
    constexpr int NS = 16;                       // steps per slice
    const int s0 = slice * NS;
    uint4 aq[NS];
    const uint2 xv = *reinterpret_cast<const uint2*>(xrow + min(256 * slice + 4 * lane, P.H - 4));
#pragma unroll
    for (int u = 0; u < NS; ++u) {
        const size_t f = (size_t)ta * ksteps + min(s0 + u, ksteps - 1);       // fragment; fp8 fragments: 8 bytes per lane, two lanes per word
        aq[u] = af[FP8 ? f * 32 + (lane >> 1) : f * 64 + lane];
    }
    xl[w][lane] = xv;
    wave_fence();
    float acc = 0.f;
#pragma unroll
    for (int u = 0; u < NS; ++u) {
        if (s0 + u < ksteps) {
            const uint4 xa = *reinterpret_cast<const uint4*>(&xl[w][4 * u + 2 * hf]);
            const uint32_t xw[4] = {xa.x, xa.y, xa.z, xa.w};
            const uint32_t aw[4] = {aq[u].x, aq[u].y, aq[u].z, aq[u].w};
            if (FP8) {
                const uint32_t d[2] = {(lane & 1) ? aw[2] : aw[0], (lane & 1) ? aw[3] : aw[1]};
#pragma unroll
                for (int j = 0; j < 4; ++j) {      // elements 2j, 2j + 1: bytes 2 (j % 2), 2 (j % 2) + 1 of word j / 2
                    const auto a2 = (j & 1) ? __builtin_amdgcn_cvt_pk_f32_fp8(d[j >> 1], true)
                                            : __builtin_amdgcn_cvt_pk_f32_fp8(d[j >> 1], false);
                    acc = fmaf(__uint_as_float(xw[j] << 16), a2[0], acc);
                    acc = fmaf(__uint_as_float(xw[j] & 0xFFFF0000u), a2[1], acc);
                }
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    acc = fmaf(__uint_as_float(xw[j] << 16), tq_half_bits_to_float((uint16_t)(aw[j] & 0xFFFF)), acc);
                    acc = fmaf(__uint_as_float(xw[j] & 0xFFFF0000u), tq_half_bits_to_float((uint16_t)(aw[j] >> 16)), acc);
                }
            }
        }
    }
    acc += __shfl_xor(acc, 32);
    if (hf == 0) red[w][col] = acc;
    __syncthreads();
    const int c = 32 * ta + (int)threadIdx.x;
    if (threadIdx.x < 32 && c < P.na) {
        float s = red[0][threadIdx.x];
#pragma unroll
        for (int i = 1; i < TQ_PRE_PART_SLICES; ++i) s += red[i][threadIdx.x];
        if (FP8) s *= tq_sig_base(P.blob, P.expert_stride, P.sec, P.fm, 0, e)[c];
        P.t[((size_t)v * P.n_parts + part) * P.na + c] = s;
    }
}

// The whole permutation of at most TQ_PERM_CHUNK assignments in ONE wavefront and one launch; with
// PRE != 0 the other workgroups of the launch compute the gate/up low-rank intermediate by assignment (1: fp16
// factors, 2: fp8 factors) or derive what the tiled kernels read beside the blob (3).
// With ROUTE the launch also does the routing (route_small; idx and w are then unused).
// (Workgroups of as many waves as a part of the pre-pass has slices; the permutation's is one wave, the others end at once.)
template <int PRE, bool ROUTE>
__global__ void __launch_bounds__(PRE == 1 || PRE == 2 ? 64 * TQ_PRE_PART_SLICES : 64) permute_small_kernel(const int32_t* __restrict__ idx, const float* __restrict__ w,
                                                           int n_assign, int E, int S, int T, int k,
                                                           int32_t* __restrict__ offsets, int32_t* __restrict__ slot_of,
                                                           int slot_stride, int32_t* __restrict__ src_of,
                                                           int32_t* __restrict__ row_token, float* __restrict__ row_w,
                                                           int32_t* __restrict__ tile_e, int32_t* __restrict__ tile_row0,
                                                           int rt_max, int32_t* __restrict__ ctrl,
                                                           int32_t* __restrict__ err_flag,
                                                           const TqBlobHeader* __restrict__ hdr, TqBlobHeader expect,
                                                           int check_blob, int32_t* __restrict__ zero_buf, int zero_n,
                                                           std::conditional_t<PRE == 3, TqPrep, TqPreByAssign> P, int tilings, TqRouteIn R,
                                                           int route_off)
{
    if constexpr (PRE == 3) {
        if (blockIdx.x > 0) {
            tq_prep_wave(P, blockIdx.x - 1, threadIdx.x);
            return;
        }
    } else if (PRE != 0 && blockIdx.x > 0) {
        if (check_blob && !blob_header_ok(hdr, expect)) return;      // a blob of another layer is not indexed
        pre_by_assign_block<PRE == 2>(P, idx, T, E, k, blockIdx.x - 1, ROUTE ? &R : nullptr);
        return;
    }
    if (threadIdx.x >= 64) return;
    if (ROUTE) {
        extern __shared__ int32_t sm_all[];
        int32_t* ridx = sm_all + route_off;
        float* rw = reinterpret_cast<float*>(ridx + TQ_PERM_CHUNK);
        route_small(R, T, E, k, ridx, rw, threadIdx.x);
        __syncthreads();
        idx = ridx;
        w = rw;
    }
    permute_small_body(idx, w, n_assign, E, S, T, k, offsets, slot_of, slot_stride, src_of, row_token, row_w, tile_e,
                       tile_row0, rt_max, ctrl, err_flag, hdr, expect, check_blob, zero_buf, zero_n, tilings);
}

}  // namespace

tq_status tqi_launch_permute(const int32_t* topk_idx, const float* topk_w, int32_t T, int32_t E, int32_t S,
                             int32_t k, int32_t* offsets, int32_t* slot_of, int32_t slot_stride,
                             int32_t* src_of, int32_t* row_token, float* row_w, int32_t* tile_e,
                             int32_t* tile_row0, int32_t rt_max, int32_t* ctrl, int32_t* err_flag,
                             int32_t* hist, int32_t nblk, const void* blob, const TqLayout* L,
                             int32_t* zero_buf, int32_t zero_n, hipStream_t stream, const TqPreByAssign* pre, int tilings,
                             const TqRouteIn* route, const TqPrep* prep)
{
    const int64_t n_assign = (int64_t)T * k;
    const unsigned n_prep = prep ? prep->n_waves : 0;
    const int64_t n_pre = pre ? (int64_t)pre->a_tot * pre->n_parts * pre->na_tiles : 0;
    if (n_pre > 0x3FFFFFFF) return TQ_ERR_UNSUPPORTED;
    TqBlobHeader expect = {};
    int check = 0;
    if (blob && L) {
        check = 1;
        expect.magic = TQ_BLOB_MAGIC; expect.version = TQ_BLOB_VERSION;
        expect.n_experts = L->E; expect.n_shared = L->S; expect.hidden = L->H; expect.ffn = L->F;
        expect.group = L->g; expect.bits = L->bits; expect.rank = L->r; expect.expert_stride = L->expert_stride;
        expect.code_words = L->cw; expect.factor_fp8 = L->fm.fp8; expect.tiles_m = L->fm.M; expect.tiles_n = L->fm.N;
    }
    const int ne = E + S;
    if (nblk == 1 && (int64_t)S * T <= 4096) {
        const int sm_words = ne + (ne + 1) + E + TQ_N_TILINGS * (ne + 1);
        const bool fused = route != nullptr;
        if (fused && !tqi_route_fusable(T, E, S, k, nblk)) return TQ_ERR_UNSUPPORTED;
        const size_t sm = ((size_t)sm_words + (fused ? 2 * TQ_PERM_CHUNK : 0)) * 4;
        const int pre_kind = n_pre > 0 ? (pre->fm.fp8 ? 2 : 1) : 0;
        const TqRouteIn R = fused ? *route : TqRouteIn{};
        const TqPreByAssign P = n_pre > 0 ? *pre : TqPreByAssign{};
#define TQ_PS(PREV, ROUTEV, P, NV)                                                                                        \
        hipLaunchKernelGGL((permute_small_kernel<PREV, ROUTEV>), dim3(1 + (unsigned)(NV)), dim3(pre_kind ? 64 * TQ_PRE_PART_SLICES : 64), sm, stream, topk_idx,  \
                           topk_w, (int)n_assign, E, S, T, k, offsets, slot_of, slot_stride, src_of, row_token, row_w,     \
                           tile_e, tile_row0, rt_max, ctrl, err_flag, (const TqBlobHeader*)blob, expect, check, zero_buf,  \
                           (int)zero_n, P, tilings, R, sm_words)
        if (n_prep > 0) {      // (a tiled path: no pre-pass by assignment)
            if (n_pre > 0) return TQ_ERR_UNSUPPORTED;
            if (fused) TQ_PS(3, true, *prep, n_prep); else TQ_PS(3, false, *prep, n_prep);
        } else if (fused) {
            if (pre_kind == 2) TQ_PS(2, true, P, n_pre); else if (pre_kind == 1) TQ_PS(1, true, P, n_pre); else TQ_PS(0, true, P, n_pre);
        } else {
            if (pre_kind == 2) TQ_PS(2, false, P, n_pre); else if (pre_kind == 1) TQ_PS(1, false, P, n_pre); else TQ_PS(0, false, P, n_pre);
        }
#undef TQ_PS
        TQ_CHECK_LAUNCH();
        return TQ_OK;
    }
    if (route) return TQ_ERR_UNSUPPORTED;      // the caller routes by itself when the single-wave permutation does not run
    if (n_pre > 0) return TQ_ERR_UNSUPPORTED;  // (at most 256 rows: always the single-wave permutation)
    const unsigned nb = (unsigned)((n_assign + TQ_PLACE_CHUNK - 1) / TQ_PLACE_CHUNK);
    const bool count_self = n_assign <= TQ_PLACE_COUNT_SELF;
    const bool scan = !count_self && (int64_t)nb * E >= TQ_PLACE_SCAN_WORDS;
    // the workspace's nblk x E words hold nb x E counts, nb flags and E totals: nblk >= 4 nb - 3 and nb >= 5 here
    if (!count_self) {
        hipLaunchKernelGGL(permute_hist_kernel, dim3(nb), dim3(TQ_PLACE_THREADS), (size_t)(E + 1) * 4, stream, topk_idx, n_assign, E,
                           hist);
        TQ_CHECK_LAUNCH();
    }
    if (scan) {
        int ep = 1;
        while (ep < E && ep < 32) ep *= 2;
        hipLaunchKernelGGL(permute_scan_kernel, dim3((E + ep - 1) / ep), dim3(TQ_SCAN_THREADS), 0, stream, hist, (int)nb, E, ep);
        TQ_CHECK_LAUNCH();
    }
    // at most 64 KB: E <= 1024 and S <= 64 at every entry point
    const size_t sm = ((size_t)E + ne + (ne + 1) + TQ_N_TILINGS * (ne + 1) + (size_t)TQ_PLACE_WAVES * E + 1) * 4;
#define TQ_PP(PREPV, P)                                                                                                     \
    hipLaunchKernelGGL(permute_place_kernel<PREPV>, dim3(nb + (n_prep + TQ_PLACE_THREADS / 64 - 1) / (TQ_PLACE_THREADS / 64)), \
                       dim3(TQ_PLACE_THREADS), sm, stream, topk_idx, topk_w, n_assign, E, S, T, k, count_self ? nullptr : hist, \
                       (int)scan, offsets, slot_of, slot_stride, src_of, row_token, row_w, tile_e, tile_row0, rt_max, ctrl, err_flag, \
                       (const TqBlobHeader*)blob, expect, check, zero_buf, (int)zero_n, tilings, (int)nb, P)
    if (n_prep > 0) TQ_PP(true, *prep); else TQ_PP(false, NoPrep{});
#undef TQ_PP
    TQ_CHECK_LAUNCH();
    return TQ_OK;
}

extern "C" tq_status tq_route(const float* logits, const float* bias, int32_t T, int32_t E, int32_t k,
                              int32_t* topk_idx, float* topk_w, void* stream)
{
    if (!logits || !topk_idx || !topk_w) return TQ_ERR_NULL;
    if (T < 0 || E < 1 || k < 1 || k > E) return TQ_ERR_SHAPE;
    if (E > 64 * kMaxPerLane || k > 64) return TQ_ERR_UNSUPPORTED;
    if (((uintptr_t)logits | (uintptr_t)topk_idx | (uintptr_t)topk_w | (uintptr_t)bias) & 3) return TQ_ERR_ALIGN;
    if (T == 0) return TQ_OK;
    const int per_lane = (E + 63) / 64;
    const dim3 grid((T + 3) / 4), block(256);
    hipStream_t st = (hipStream_t)stream;
    const dim3 grid16((T + 15) / 16);
    // rows of 16 lanes up to 16 selections and 256 experts; beyond, a wave per token with as many scores per lane as it needs
    // (8192 tokens, 32 selections of 64 experts: 47.8 us with one, 55.0 with room for four; of 128: 49.1 with two, 54.9)
    if (k <= 16 && E <= 64) hipLaunchKernelGGL(route_row_kernel<4>, grid16, block, 0, st, logits, bias, T, E, k, topk_idx, topk_w);
    else if (k <= 16 && E <= 128) hipLaunchKernelGGL(route_row_kernel<8>, grid16, block, 0, st, logits, bias, T, E, k, topk_idx, topk_w);
    else if (k <= 16 && E <= 256) hipLaunchKernelGGL(route_row_kernel<16>, grid16, block, 0, st, logits, bias, T, E, k, topk_idx, topk_w);
    else if (per_lane == 1) hipLaunchKernelGGL(route_kernel<1>, grid, block, 0, st, logits, bias, T, E, k, topk_idx, topk_w);
    else if (per_lane == 2) hipLaunchKernelGGL(route_kernel<2>, grid, block, 0, st, logits, bias, T, E, k, topk_idx, topk_w);
    else if (per_lane <= 4) hipLaunchKernelGGL(route_kernel<4>, grid, block, 0, st, logits, bias, T, E, k, topk_idx, topk_w);
    else hipLaunchKernelGGL(route_kernel<kMaxPerLane>, grid, block, 0, st, logits, bias, T, E, k, topk_idx, topk_w);
    TQ_CHECK_LAUNCH();
    return TQ_OK;
}

extern "C" size_t tq_permute_workspace_size(int32_t T, int32_t E, int32_t k)
{
    if (T < 0 || E < 1 || k < 1) return 0;
    int64_t nblk = ((int64_t)T * k + TQ_PERM_CHUNK - 1) / TQ_PERM_CHUNK;
    if (nblk < 1) nblk = 1;
    return tq_align256((size_t)nblk * E * 4);
}

extern "C" tq_status tq_permute(const int32_t* topk_idx, int32_t T, int32_t E, int32_t k, int32_t* offsets,
                                int32_t* slot_of, int32_t* src_of, int32_t* err_flag, void* workspace,
                                size_t workspace_bytes, void* stream)
{
    if (!topk_idx || !offsets || !slot_of || !src_of || !workspace) return TQ_ERR_NULL;
    if (T < 0 || E < 1 || E > 1024 || k < 1 || k > E) return TQ_ERR_SHAPE;
    if (workspace_bytes < tq_permute_workspace_size(T, E, k)) return TQ_ERR_WORKSPACE;
    if (((uintptr_t)topk_idx | (uintptr_t)offsets | (uintptr_t)slot_of | (uintptr_t)src_of |
         (uintptr_t)err_flag | (uintptr_t)workspace) & 3)
        return TQ_ERR_ALIGN;
    int64_t nblk = ((int64_t)T * k + TQ_PERM_CHUNK - 1) / TQ_PERM_CHUNK;
    if (nblk < 1) nblk = 1;     // T == 0 runs the single-wave kernel with nothing to place: offsets become all zero
    return tqi_launch_permute(topk_idx, nullptr, T, E, 0, k, offsets, slot_of, k, src_of, nullptr, nullptr,
                              nullptr, nullptr, 0, nullptr, err_flag, (int32_t*)workspace, (int32_t)nblk, nullptr,
                              nullptr, nullptr, 0, (hipStream_t)stream);
}
