// Gating top-k, per-expert batching and gate-weighted combine for gfx950.
//
// route  : G = next power of two >= E lanes of a wavefront hold one token's
//          logits; k rounds of a butterfly arg-max (value desc, index asc)
//          pick the experts; the softmax over the k winners is fp32.
// permute: a stable counting sort of the T*k slots keyed on the expert.  Every workgroup
//          counts all slots and places its own (ranks: wavefront ballots, lanes below me
//          with my expert), so the order inside an expert segment is the slot order and
//          the result is unique.
// combine: y[t] = sum_j w[t,j] * yg[inv_perm[t*k+j]], float4 lanes along d.
#include <type_traits>

#include "moe_internal.h"
#include "moe_gate_wave.h"

// ------------------------------------------------------------------ route ----

// The contest for the token whose logits the group's G lanes hold (lane gl: expert e = gl with logit v, or -inf and
// INT_MAX): returns the weight of the group's gl-th winner, my_i, for lanes gl < k.
template <int G>
__device__ __forceinline__ float route_token(float v, int e, int gl, int k, int& my_i) {
    float my_v = 0.f, top_v = 0.f;
    my_i = 0;
    for (int j = 0; j < k; j++) {
        float bv = v;
        int be = e;
#pragma unroll
        for (int m = 1; m < G; m <<= 1) {
            float ov = __shfl_xor(bv, m, 64);
            int oe = __shfl_xor(be, m, 64);
            if (ov > bv || (ov == bv && oe < be)) {
                bv = ov;
                be = oe;
            }
        }
        if (j == 0) top_v = bv;
        if (gl == j) {
            my_v = bv;
            my_i = be;
        }
        if (e == be) {  // the winner leaves the contest
            v = -INFINITY;
            e = 0x7fffffff;
        }
    }
    float u = (gl < k) ? expf(my_v - top_v) : 0.f;
    float s = u;
#pragma unroll
    for (int m = 1; m < G; m <<= 1) s += __shfl_xor(s, m, 64);
    return u / s;
}

template <int G>
__global__ __launch_bounds__(256) void route_kernel(const float* __restrict__ logits, int T, int E,
                                                    int k, int32_t* __restrict__ idx,
                                                    float* __restrict__ weights) {
    const int tid = blockIdx.x * 256 + threadIdx.x;
    const int t = tid / G;
    const int gl = tid % G;  // lane inside the token's group = expert id it holds
    const bool live = (t < T);
    float v = -INFINITY;
    int e = 0x7fffffff;
    if (live && gl < E) {
        v = logits[(size_t)t * E + gl];
        e = gl;
    }
    int my_i;
    const float w = route_token<G>(v, e, gl, k, my_i);
    if (live && gl < k) {
        idx[(size_t)t * k + gl] = my_i;
        weights[(size_t)t * k + gl] = w;
    }
}

int moe_route_launch(const float* logits, int T, int E, int k, int32_t* idx, float* weights,
                     hipStream_t s) {
    int G = 1;
    while (G < E) G <<= 1;
    if (G < k) G = 8;  // cannot happen (k <= E); keeps lanes gl < k inside the group
    const int tok_per_block = 256 / G;
    const unsigned grid = (unsigned)((T + tok_per_block - 1) / tok_per_block);
#define ROUTE_CASE(g)                                                                         \
    case g:                                                                                   \
        hipLaunchKernelGGL(route_kernel<g>, dim3(grid), dim3(256), 0, s, logits, T, E, k, idx, \
                           weights);                                                          \
        break;
    switch (G) {
        ROUTE_CASE(1)
        ROUTE_CASE(2)
        ROUTE_CASE(4)
        ROUTE_CASE(8)
        ROUTE_CASE(16)
        ROUTE_CASE(32)
        ROUTE_CASE(64)
        default:
            return MOE_ERR_INVALID_ARG;
    }
#undef ROUTE_CASE
    return moe_launch_status();
}

// ---------------------------------------------------------------- permute ----

#define PERM_THREADS 1024
#define PERM_WAVES (PERM_THREADS / 64)

// Index part of the batching for the few slots of the fused front ends (gate_small_kernel), run
// by every workgroup of 1024 threads for itself, so that each can then gather its share of rows.
// Outputs are written only when `write` is set.  Returns through LDS: s_off.
__device__ void permute_indices(const int32_t* __restrict__ idx, int N, int E,
                                int32_t* __restrict__ counts, int32_t* __restrict__ offsets,
                                int32_t* __restrict__ perm, int32_t* __restrict__ inv_perm,
                                bool write, int* s_cnt /*[64]*/, int* s_off /*[65]*/,
                                int* s_wave /*[PERM_WAVES][64]*/, int* s_pos /*[1024] or null*/) {
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    if (tid < MOE_MAX_E) s_cnt[tid] = 0;
    __syncthreads();
    for (int p = tid; p < N; p += PERM_THREADS) {
        int e = idx[p];
        e = e < 0 ? 0 : (e >= E ? E - 1 : e);
        atomicAdd(&s_cnt[e], 1);
    }
    __syncthreads();
    if (tid == 0) {
        int run = 0;
        for (int e = 0; e < E; e++) {
            s_off[e] = run;
            run += s_cnt[e];
        }
        s_off[E] = run;
    }
    __syncthreads();
    if (write) {
        if (tid < E) counts[tid] = s_cnt[tid];
        if (tid <= E) offsets[tid] = s_off[tid];
    }
    // s_cnt now becomes the running number of slots already placed per expert.
    __syncthreads();
    if (tid < MOE_MAX_E) s_cnt[tid] = 0;
    __syncthreads();
    const unsigned long long below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    for (int base = 0; base < N; base += PERM_THREADS) {
        const int p = base + tid;
        int e = -1;
        if (p < N) {
            e = idx[p];
            e = e < 0 ? 0 : (e >= E ? E - 1 : e);
        }
        int rank = 0;
        for (int ee = 0; ee < E; ee++) {
            unsigned long long m = __ballot(e == ee);
            if (e == ee) rank = __popcll(m & below);
            if (lane == 0) s_wave[wave * MOE_MAX_E + ee] = __popcll(m);
        }
        __syncthreads();
        if (tid < E) {
            int run = s_cnt[tid];
            for (int w = 0; w < PERM_WAVES; w++) {
                int c = s_wave[w * MOE_MAX_E + tid];
                s_wave[w * MOE_MAX_E + tid] = run;
                run += c;
            }
            s_cnt[tid] = run;
        }
        __syncthreads();
        if (p < N) {
            const int pos = s_off[e] + s_wave[wave * MOE_MAX_E + e] + rank;
            if (write) {
                perm[pos] = p;
                inv_perm[p] = pos;
            }
            if (s_pos) s_pos[p] = pos;
        }
        __syncthreads();
    }
}

// moe_permute: one launch.  Workgroup b takes the slots of `tpw` consecutive tokens.  It counts
// the experts of all N slots (LDS histograms, one per wave, slots before its own apart from the
// rest), which gives it the segment offsets and the positions of its own slots without waiting
// for another workgroup; ranks inside a group of 64 slots are ballots.  GATHER: then its waves
// copy their tokens' rows, each row read once and stored at its k positions.
// Bound: reading idx from L2 in every workgroup (N * 4 bytes each), then the row copy.  One
// workgroup for all N slots (and a second launch that read every row k times) took 15 + 21 us at
// 4096 tokens, k = 2, 8 KiB rows, and 14 us for the indices of 300 tokens, k = 6, 64 experts;
// this one launch 18.5 and 5 us.  Routing, batching and combine together: 4096 tokens, k = 2, pass after pass over three
// sets of buffers 80.7 -> 60 us (a single pass on buffers that were not used before gains less, 70.5 -> 68); 8192 tokens, k
// = 6, 64 experts, 4 KiB rows 452 -> 173 us on the same buffers.
#define PM_THREADS 512
#define PM_WAVES (PM_THREADS / 64)
#define PM_MAX_SLOTS 1024  // slots of a workgroup whose positions are kept for the row copy
#define PM_EARLY_SLOTS 4096
static_assert(PM_EARLY_SLOTS >= PM_THREADS * 4, "at least one round of requests");

// A wave's part of a row: 8 KiB of loads in flight, stored to k rows of xg.  pos(j): row of copy j.
// STREAM: past L2 (the rows are read once), from 16 rows of a workgroup (two per wave; more than 15 tokens per CU).  No
// line in the times there: with 9..15 rows the differences are the same.  They lie in where the rows are.  In
// memory: 8 KiB rows, k = 2, 3841 tokens 21.8 -> 18.7 us, 4096 24.8 -> 19.7, 16 KiB rows 43.2 -> 41.8; just written by another
// kernel: even (17.5, 32 us), where rows and copies exceed the last-level cache 71 -> 66; read by this call last time, with
// nothing between: 4096 tokens 18.0 -> 18.2, 8192 34.5 -> 36.9, 16 KiB rows 31.9 -> 34.2, k = 1 21.5 -> 24.8.  128-byte
// rows even.  Gating, batching and combine with buffers that change, 4096 tokens 64 -> 60 us, with the residual add that
// reads x and y next 91 -> 87.
template <bool STREAM>
__device__ __forceinline__ void load_row(const u32x4_t* __restrict__ src, int row_chunks, int c0, u32x4_t (&v)[8]) {
#pragma unroll
    for (int u = 0; u < 8; u++) {  // past the end of the row: its last chunk, not stored
        const u32x4_t* p = src + (c0 + u * 64 < row_chunks ? c0 + u * 64 : row_chunks - 1);
        v[u] = STREAM ? __builtin_nontemporal_load(p) : *p;
    }
}
template <class POS>
__device__ __forceinline__ void store_row_k(const u32x4_t (&v)[8], u32x4_t* __restrict__ xg, int row_chunks, int k,
                                            int c0, POS pos) {
    for (int j = 0; j < k; j++) {
        u32x4_t* dst = xg + (size_t)pos(j) * row_chunks;
#pragma unroll
        for (int u = 0; u < 8; u++)
            if (c0 + u * 64 < row_chunks) dst[c0 + u * 64] = v[u];
    }
}
// One row from chunk c0 (of this lane) on, copied by a wave to k rows of xg, the row read once.
template <bool STREAM, class POS>
__device__ __forceinline__ void copy_row_k(const u32x4_t* __restrict__ src, u32x4_t* __restrict__ xg,
                                           int row_chunks, int k, int c0, POS pos) {
    for (; c0 < row_chunks; c0 += 64 * 8) {
        u32x4_t v[8];
        load_row<STREAM>(src, row_chunks, c0, v);
        store_row_k(v, xg, row_chunks, k, c0, pos);
    }
}

template <bool GATHER, bool EARLY, bool STREAM>
__global__ __launch_bounds__(PM_THREADS) void permute_kernel(
    const int32_t* __restrict__ idx, int N, int E, int k, int tpw, const u32x4_t* __restrict__ x,
    int row_chunks /* 16-byte chunks per row */, int32_t* __restrict__ counts,
    int32_t* __restrict__ offsets, int32_t* __restrict__ perm, int32_t* __restrict__ inv_perm,
    u32x4_t* __restrict__ xg) {
    __shared__ int s_hist[PM_WAVES][2][MOE_MAX_E];  // [wave][slots before mine, the rest][expert]
    __shared__ int s_next[MOE_MAX_E];               // next free position per expert
    __shared__ int s_pos[GATHER ? PM_MAX_SLOTS : 1];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // (a wave clears and fills its own histogram only: its LDS operations are in order)
    s_hist[wave][0][lane] = 0;
    s_hist[wave][1][lane] = 0;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const int slot0 = blockIdx.x * tpw * k;  // (grid * tpw tokens: below 2^25 slots)
    const int slots = (N - slot0) < tpw * k ? (N - slot0) : tpw * k;
    auto expert = [&](int e) { return e < 0 ? 0 : (e >= E ? E - 1 : e); };
    // wave 0's first group of its own slots, requested before the count instead of behind it
    const int own = (wave == 0 && lane < slots) ? idx[slot0 + lane] : 0;
    auto count = [&](int p, const int4& v) {  // slots p .. p+3
        const int e[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int q = 0; q < 4; q++)
            if (p + q < N) atomicAdd(&s_hist[wave][p + q < slot0 ? 0 : 1][expert(e[q])], 1);
    };
    auto load4 = [&](int p) -> int4 {
        if (p + 4 <= N) return *(const int4*)(idx + p);
        int4 v;
        v.x = p < N ? idx[p] : 0;
        v.y = p + 1 < N ? idx[p + 1] : 0;
        v.z = p + 2 < N ? idx[p + 2] : 0;
        v.w = 0;
        return v;
    };
    const int tokens = slots / k, t0 = slot0 / k;
    u32x4_t r0[8], r1[8];
    int p = tid * 4;
    // EARLY, from PM_EARLY_SLOTS slots on: the requests for slots first (up to PM_EARLY rounds of the
    // workgroup), then the first rows to be copied, then the count, which is done while the rows come.  4096
    // tokens, k = 2, 8 KiB rows 20.4 -> 18.2 us, 16 KiB rows of 8192 tokens 86 -> 81; fewer slots are counted before
    // rows could come (100 tokens, 16 KiB rows 4.6 -> 5.0, 1000 tokens 10.5 -> 10.9).
    constexpr int PM_EARLY = 4;
    if (EARLY) {
        const int rounds = N / (PM_THREADS * 4);  // (uniform, at least 1)
        int4 first[PM_EARLY];
#pragma unroll
        for (int i = 0; i < PM_EARLY; i++)
            if (i < rounds) first[i] = *(const int4*)(idx + p + i * PM_THREADS * 4);
        if (wave < tokens) load_row<STREAM>(x + (size_t)(t0 + wave) * row_chunks, row_chunks, lane, r0);
        if (wave + PM_WAVES < tokens) load_row<STREAM>(x + (size_t)(t0 + wave + PM_WAVES) * row_chunks, row_chunks, lane, r1);
#pragma unroll
        for (int i = 0; i < PM_EARLY; i++)
            if (i < rounds) count(p + i * PM_THREADS * 4, first[i]);
        p += (rounds < PM_EARLY ? rounds : PM_EARLY) * PM_THREADS * 4;
    }
    for (; p < N; p += PM_THREADS * 4) count(p, load4(p));
    __syncthreads();
    if (wave == 0) {
        int before = 0, rest = 0;
        for (int w = 0; w < PM_WAVES; w++) {
            before += s_hist[w][0][lane];
            rest += s_hist[w][1][lane];
        }
        const int cnt = before + rest;  // 0 for lanes >= E
        int inc = cnt;
#pragma unroll
        for (int dlt = 1; dlt < 64; dlt <<= 1) {
            const int v = __shfl_up(inc, dlt, 64);
            if (lane >= dlt) inc += v;
        }
        if (blockIdx.x == 0) {
            if (lane < E) {
                counts[lane] = cnt;
                offsets[lane] = inc - cnt;
            }
            if (lane == E - 1) offsets[E] = inc;
        }
        s_next[lane] = inc - cnt + before;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        // positions, 64 slots at a time: rank among the group's lower slots of the same expert
        const unsigned long long below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
        for (int g = 0; g < slots; g += 64) {
            const int p = slot0 + g + lane;
            const bool live = g + lane < slots;
            const int e = live ? expert(g == 0 ? own : idx[p]) : 0;
            unsigned long long same = __ballot(live);
#pragma unroll
            for (int b = 0; b < 6; b++) {  // E <= 64
                const unsigned long long m = __ballot((e >> b) & 1);
                same &= ((e >> b) & 1) ? m : ~m;
            }
            const int rank = __popcll(same & below);
            int pos = 0;
            if (live) pos = s_next[e] + rank;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            if (live) {
                if (rank == 0) s_next[e] = pos + __popcll(same);
                perm[pos] = p;
                inv_perm[p] = pos;
                if (GATHER) s_pos[g + lane] = pos;
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
    }
    if (!GATHER) return;
    __syncthreads();
    for (int t = wave; t < tokens; t += PM_WAVES) {
        const u32x4_t* src = x + (size_t)(t0 + t) * row_chunks;
        auto pos = [&](int j) { return s_pos[t * k + j]; };
        const bool early = EARLY && t < 2 * PM_WAVES;
        if (early && t < PM_WAVES) store_row_k(r0, xg, row_chunks, k, lane, pos);
        else if (early) store_row_k(r1, xg, row_chunks, k, lane, pos);
        copy_row_k<STREAM>(src, xg, row_chunks, k, early ? lane + 64 * 8 : lane, pos);
    }
}

// xg[inv_perm[t*k+j],:] = x[t,:]: the row copy on its own, one wave per token (calls whose
// workgroups hold more slots than PM_MAX_SLOTS).
__global__ __launch_bounds__(256) void gather_rows_kernel(const int32_t* __restrict__ inv_perm, int T,
                                                          int k, const u32x4_t* __restrict__ x,
                                                          int row_chunks,
                                                          u32x4_t* __restrict__ xg) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int t = blockIdx.x * 4 + wave; t < T; t += gridDim.x * 4)
        copy_row_k<false>(x + (size_t)t * row_chunks, xg, row_chunks, k, lane,
                   [&](int j) { return inv_perm[(size_t)t * k + j]; });
}

int moe_permute_launch(const int32_t* idx, int T, int E, int k, const void* x, int d,
                       moe_dtype_t x_dtype, int32_t* counts, int32_t* offsets, int32_t* perm,
                       int32_t* inv_perm, void* xg, hipStream_t s) {
    const int N = T * k;
    const int row_chunks = (int)(((size_t)d * (x_dtype == MOE_BF16 ? 2 : 4)) / 16);
    // one workgroup per CU at most: every one counts all N slots
    const int cus = moe_num_cus();
    const int tpw = T > cus ? (T + cus - 1) / cus : 1;
    const unsigned grid = T > 0 ? (unsigned)((T + tpw - 1) / tpw) : 1u;
    const bool fused = x != nullptr && (long long)tpw * k <= PM_MAX_SLOTS;
    if (fused) {
        auto* kernel = N < PM_EARLY_SLOTS ? permute_kernel<true, false, false>
                       : tpw < 2 * PM_WAVES ? permute_kernel<true, true, false> : permute_kernel<true, true, true>;
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(PM_THREADS), 0, s, idx, N, E, k, tpw, (const u32x4_t*)x, row_chunks,
                           counts, offsets, perm, inv_perm, (u32x4_t*)xg);
    } else
        hipLaunchKernelGGL((permute_kernel<false, false, false>), dim3(grid), dim3(PM_THREADS), 0, s, idx, N, E, k, tpw,
                           (const u32x4_t*)nullptr, 0, counts, offsets, perm, inv_perm, (u32x4_t*)nullptr);
    if (moe_launch_status() != MOE_OK) return MOE_ERR_HIP;
    if (x != nullptr && !fused) {
        hipLaunchKernelGGL(gather_rows_kernel, dim3((unsigned)(cus * 8)), dim3(256), 0, s, inv_perm, T, k,
                           (const u32x4_t*)x, row_chunks, (u32x4_t*)xg);
        return moe_launch_status();
    }
    return MOE_OK;
}

// Routing and batching of a few slots in one launch, for moe_layer: every workgroup routes all tokens (G lanes each) and
// places all slots for itself, writes its own tokens' idx and weights and copies their rows; workgroup 0 writes the
// batch's indices.  Same values as the two calls.  Launches and latency are everything at these sizes (the host
// issues them more slowly than they run): all-fp32 layer of 16 tokens, d = 256, f = 512, 8 experts, call after call 36.2..37.1
// -> 31.4..34.1 us by the host's speed, with four launches for five.  The limit is what one wave can place (8 groups of 64
// slots), a token per CU.
#define RP_MAX_SLOTS 512
template <int G>
__global__ __launch_bounds__(PM_THREADS) void route_permute_kernel(
    const float* __restrict__ logits, int T, int EL /* logits of a token */, int E, int k, const u32x4_t* __restrict__ x,
    int row_chunks, int32_t* __restrict__ idx, float* __restrict__ weights, int32_t* __restrict__ counts,
    int32_t* __restrict__ offsets, int32_t* __restrict__ perm, int32_t* __restrict__ inv_perm, u32x4_t* __restrict__ xg) {
    __shared__ int s_idx[RP_MAX_SLOTS], s_pos[RP_MAX_SLOTS];
    __shared__ int s_next[MOE_MAX_E];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int N = T * k, own = blockIdx.x;  // one token per workgroup
    // the row that wave 1 will copy, requested first
    u32x4_t row[8];
    const u32x4_t* src = x + (size_t)own * row_chunks;
    if (wave == 1) load_row<false>(src, row_chunks, lane, row);
    const int gl = tid % G;
    for (int t0 = 0; t0 < T; t0 += PM_THREADS / G) {
        const int t = t0 + tid / G;
        float v = -INFINITY;
        int e = 0x7fffffff;
        if (t < T && gl < EL) {
            v = logits[(size_t)t * EL + gl];
            e = gl;
        }
        int my_i;
        const float w = route_token<G>(v, e, gl, k, my_i);
        if (t < T && gl < k) {
            s_idx[t * k + gl] = my_i;
            if (t == own) {
                idx[(size_t)t * k + gl] = my_i;
                weights[(size_t)t * k + gl] = w;
            }
        }
    }
    if (tid < MOE_MAX_E) s_next[tid] = 0;
    __syncthreads();
    if (wave == 0) {
        // places inside the expert's segment, 64 slots at a time, as in permute_kernel
        const unsigned long long below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
        for (int g = 0; g < N; g += 64) {
            const bool live = g + lane < N;
            int e = live ? s_idx[g + lane] : 0;
            e = e < 0 ? 0 : (e >= E ? E - 1 : e);  // (NaN logits: no id, and no access out of range)
            unsigned long long same = __ballot(live);
#pragma unroll
            for (int b = 0; b < 6; b++) {  // E <= 64
                const unsigned long long m = __ballot((e >> b) & 1);
                same &= ((e >> b) & 1) ? m : ~m;
            }
            const int rank = __popcll(same & below);
            int at = 0;
            if (live) at = s_next[e] + rank;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            if (live) {
                if (rank == 0) s_next[e] = at + __popcll(same);
                s_idx[g + lane] = e;
                s_pos[g + lane] = at;
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
        const int cnt = s_next[lane];  // 0 for lanes >= E
        int inc = cnt;
#pragma unroll
        for (int dlt = 1; dlt < 64; dlt <<= 1) {
            const int v = __shfl_up(inc, dlt, 64);
            if (lane >= dlt) inc += v;
        }
        __builtin_amdgcn_wave_barrier();
        s_next[lane] = inc - cnt;
        if (own == 0) {
            if (lane < E) {
                counts[lane] = cnt;
                offsets[lane] = inc - cnt;
            }
            if (lane == E - 1) offsets[E] = inc;
        }
    }
    __syncthreads();
    for (int p = tid; p < N; p += PM_THREADS) {
        const int pos = s_next[s_idx[p]] + s_pos[p];
        if (own == 0) {
            perm[pos] = p;
            inv_perm[p] = pos;
        }
    }
    if (wave != 1) return;
    auto pos = [&](int j) { return s_next[s_idx[own * k + j]] + s_pos[own * k + j]; };
    store_row_k(row, xg, row_chunks, k, lane, pos);
    copy_row_k<false>(src, xg, row_chunks, k, lane + 64 * 8, pos);
}

// Every workgroup routes all tokens, 512 / G at a time, where route_kernel has workgroups of their own for them: the extra
// passes cost k * log2(G) exchanges between lanes each.
// Measured, route + permute (and the time between them, about 1 us, and 2-3 us of the host's for the launch) -> this:
// 16 tokens, 8 experts, k = 2 2.1 + 3.6 -> 4.3 us, 64 tokens 2.4 + 3.6 -> 4.6; 6 exchanges more (128 tokens) 2.6 + 3.6 -> 6.2, 12
// (192) 3.1 + 3.6 -> 7.8, 18 (256) 3.0 + 3.6 -> 9.9; 20 (32 tokens, 32 experts, k = 4) 3.8 + 3.8 -> 8.7; 36 (16 tokens, 64 experts, k =
// 6) 5.3 + 4.0 -> 12.3; 252 (64 of them) 5.8 + 4.0 -> 36.
#define RP_MAX_EXTRA 12
static int rp_lanes(int EL) {
    int G = 1;
    while (G < EL) G <<= 1;
    return G;
}
bool moe_route_permute_rows_supported(int T, int EL, int k) {
    if (T < 1 || T * k > RP_MAX_SLOTS || T > moe_num_cus()) return false;
    const int G = rp_lanes(EL), passes = (T * G + PM_THREADS - 1) / PM_THREADS;
    int log2G = 0;
    while ((1 << log2G) < G) log2G++;
    return (passes - 1) * k * log2G <= RP_MAX_EXTRA;
}

int moe_route_permute_rows_launch(const float* logits, int T, int EL, int E, int k, const void* x, int d,
                                  moe_dtype_t x_dtype, int32_t* idx, float* weights, int32_t* counts, int32_t* offsets,
                                  int32_t* perm, int32_t* inv_perm, void* xg, hipStream_t s) {
    const int row_chunks = (int)(((size_t)d * (x_dtype == MOE_BF16 ? 2 : 4)) / 16);
    const int G = rp_lanes(EL);
#define RP_CASE(g)                                                                                                   \
    case g:                                                                                                          \
        hipLaunchKernelGGL(route_permute_kernel<g>, dim3((unsigned)T), dim3(PM_THREADS), 0, s, logits, T, EL, E, k,  \
                           (const u32x4_t*)x, row_chunks, idx, weights, counts, offsets, perm, inv_perm, (u32x4_t*)xg); \
        break;
    switch (G) {
        RP_CASE(1)
        RP_CASE(2)
        RP_CASE(4)
        RP_CASE(8)
        RP_CASE(16)
        RP_CASE(32)
        RP_CASE(64)
        default:
            return MOE_ERR_INVALID_ARG;
    }
#undef RP_CASE
    return moe_launch_status();
}

// ---------------------------------------------------------------- combine ----

// STREAM: y is larger than the L2 caches (32 MiB in all), so the rows, read once, go past them.  A program's pass of
// gating, batching and combine and the RMSNorm that reads y next, d = 4096, k = 2, buffers that change: 2100 tokens 58.0
// us either way, 3000 74.5 -> 72.0, 4096 96.4 -> 90.1, 8192 206 -> 173; the same rows combined again and again, which
// the caches then hold, 50.4 -> 53.7, 63.8 -> 66.4, 91.4 -> 85.5, 206 -> 170.  y itself stays where its next reader finds
// it: stored past L2 the pass is faster (4096 tokens 59.8 -> 55.7) and the reader slower by more (90.1 -> 99.8 in all).
#define COMBINE_STREAM_BYTES ((size_t)32 << 20)
template <bool STREAM>
__global__ __launch_bounds__(256) void combine_kernel(const float4* __restrict__ yg,
                                                      const int32_t* __restrict__ inv_perm,
                                                      const float* __restrict__ weights, int T,
                                                      int k, int row_chunks /* d/4 */,
                                                      float4* __restrict__ y) {
    const int t = blockIdx.y;
    const int c = blockIdx.x * 256 + threadIdx.x;
    if (t >= T || c >= row_chunks) return;
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int j = 0; j < k; j++) {
        const float w = weights[(size_t)t * k + j];
        const float4* row = yg + (size_t)inv_perm[(size_t)t * k + j] * row_chunks;
        const float4 v = STREAM ? __builtin_bit_cast(float4, __builtin_nontemporal_load((const f32x4_t*)row + c)) : row[c];
        acc.x += w * v.x;
        acc.y += w * v.y;
        acc.z += w * v.z;
        acc.w += w * v.w;
    }
    y[(size_t)t * row_chunks + c] = acc;
}

int moe_combine_launch(const float* yg, const int32_t* inv_perm, const float* weights, int T, int k,
                       int d, float* y, hipStream_t s) {
    const int row_chunks = d / 4;
    dim3 grid((unsigned)((row_chunks + 255) / 256), (unsigned)T);
    auto* kernel = (size_t)T * d * sizeof(float) > COMBINE_STREAM_BYTES ? combine_kernel<true> : combine_kernel<false>;
    // gridDim.y is limited to 65535: walk T in slabs
    for (int t0 = 0; t0 < T; t0 += 65535) {
        const int tn = (T - t0) < 65535 ? (T - t0) : 65535;
        grid.y = (unsigned)tn;
        hipLaunchKernelGGL(kernel, grid, dim3(256), 0, s, (const float4*)yg,
                           inv_perm + (size_t)t0 * k, weights + (size_t)t0 * k, tn, k, row_chunks,
                           (float4*)(y + (size_t)t0 * d));
    }
    return moe_launch_status();
}

// ------------------------------------------------- stack support kernels ----

// Sum over the wave's 64 lanes, in every lane, without the LDS: inside a row of 16 lanes by DPP
// (neighbours, pairs, then the mirrored half and the mirrored row), across rows by the two lane
// swaps.  (__shfl_xor goes through the LDS, 108 times per wave and 16 waves per CU: with it, and with
// the sums of 16 experts where there are 8, norm_logits_kernel took 13.7 us at 512 tokens in a stack of
// layers, now 10.6.)
__device__ __forceinline__ float wave_sum(float v) {
    auto dpp = [](float a, auto ctrl) {
        return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, a), decltype(ctrl)::value,
                                                                     0xF, 0xF, true));
    };
    v += dpp(v, std::integral_constant<int, 0xB1>{});   // quad_perm 1,0,3,2
    v += dpp(v, std::integral_constant<int, 0x4E>{});   // quad_perm 2,3,0,1
    v += dpp(v, std::integral_constant<int, 0x141>{});  // row_half_mirror
    v += dpp(v, std::integral_constant<int, 0x140>{});  // row_mirror
    const auto a = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, v), __builtin_bit_cast(unsigned, v),
                                                    false, false);
    v = __builtin_bit_cast(float, (unsigned)a[0]) + __builtin_bit_cast(float, (unsigned)a[1]);
    const auto b = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, v), __builtin_bit_cast(unsigned, v),
                                                    false, false);
    return __builtin_bit_cast(float, (unsigned)b[0]) + __builtin_bit_cast(float, (unsigned)b[1]);
}

__device__ __forceinline__ float block_sum_256(float v, float* s_red /*[4]*/) {
    v = wave_sum(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) s_red[threadIdx.x >> 6] = v;
    __syncthreads();
    return s_red[0] + s_red[1] + s_red[2] + s_red[3];
}

__global__ __launch_bounds__(256) void rmsnorm_kernel(const float* __restrict__ x, int d, float eps,
                                                      float* __restrict__ h) {
    __shared__ float s_red[4];
    const float* row = x + (size_t)blockIdx.x * d;
    float ss = 0.f;
    for (int r = threadIdx.x; r < d; r += 256) ss += row[r] * row[r];
    ss = block_sum_256(ss, s_red);
    const float inv = 1.0f / sqrtf(ss / (float)d + eps);
    float* out = h + (size_t)blockIdx.x * d;
    for (int r = threadIdx.x; r < d; r += 256) out[r] = row[r] * inv;
}

// One workgroup per token; thread r-strided partial sums for all E logits.
__global__ __launch_bounds__(256) void router_logits_kernel(const float* __restrict__ h,
                                                            const float* __restrict__ w_gate, int d,
                                                            int E, float* __restrict__ logits) {
    __shared__ float s_red[4];
    const float* row = h + (size_t)blockIdx.x * d;
    for (int e0 = 0; e0 < E; e0 += 8) {
        float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        const int ne = (E - e0) < 8 ? (E - e0) : 8;
        for (int r = threadIdx.x; r < d; r += 256) {
            const float hv = row[r];
            const float* wr = w_gate + (size_t)r * E + e0;
#pragma unroll
            for (int j = 0; j < 8; j++)
                if (j < ne) acc[j] += hv * wr[j];
        }
#pragma unroll
        for (int j = 0; j < 8; j++) {
            const float tot = block_sum_256(acc[j], s_red);
            if (j < ne && threadIdx.x == 0) logits[(size_t)blockIdx.x * E + e0 + j] = tot;
        }
    }
}

__global__ __launch_bounds__(256) void residual_add_kernel(float4* __restrict__ x,
                                                           const float4* __restrict__ y,
                                                           size_t n4) {
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n4; i += (size_t)gridDim.x * 256) {
        float4 a = x[i];
        const float4 b = y[i];
        a.x += b.x;
        a.y += b.y;
        a.z += b.z;
        a.w += b.w;
        x[i] = a;
    }
}

int moe_rmsnorm_launch(const float* x, int T, int d, float eps, float* h, hipStream_t s) {
    hipLaunchKernelGGL(rmsnorm_kernel, dim3((unsigned)T), dim3(256), 0, s, x, d, eps, h);
    return moe_launch_status();
}

int moe_router_logits_launch(const float* h, const float* w_gate, int T, int d, int E,
                             float* logits, hipStream_t s) {
    hipLaunchKernelGGL(router_logits_kernel, dim3((unsigned)T), dim3(256), 0, s, h, w_gate, d, E,
                       logits);
    return moe_launch_status();
}

int moe_residual_add_launch(float* x, const float* y, int T, int d, hipStream_t s) {
    const size_t n4 = (size_t)T * d / 4;
    size_t blocks = (n4 + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(residual_add_kernel, dim3((unsigned)blocks), dim3(256), 0, s, (float4*)x,
                       (const float4*)y, n4);
    return moe_launch_status();
}

// --------------------------------------------- fused gate for decode-sized T ----
// One launch for the whole front end of a decode step (T <= 16 tokens): optional
// RMS normalisation + router logits, top-k routing, per-expert batching and the
// row gather.  Every workgroup recomputes the (tiny) routing state in LDS;
// workgroup 0 writes the index outputs; the workgroups share the row gather.
#define GATE_MAX_T 16       // tokens the fused gate handles
#define GATE_NORM_MAX_T 4   // ... when it also normalises and computes the router logits
#define GATE_MAX_E 16
// Partial sums of one thread for the fused RMSNorm + router: rows r = tid + i * STRIDE.
// TT = tokens handled (compile-time bound on T), UNR = rows whose loads are in flight together.
// The pending combine + residual of the block before (COMB): the row values are
//   x[t,r] + sum_j w_prev[t,j] * yg_prev[pos_prev[t,j], r]
// in the arithmetic of combine_residual_kernel.
struct GatePrev {
    const float* yg;   // [P][N_prev, d] (global): the reduction parts of the block before,
                       // added in part order (P = 1: its plain output)
    const int* pos;    // [T * k] rows of yg (inv_perm of the block before)
    const float* w;    // [T * k] gate weights of the block before
    int k;
    int P;
    size_t pstride;    // floats between two parts
};

#define GATE_MAX_PARTS 4  // reduction parts of the block before that the seam kernel adds

// PMAX: compile-time bound on pv.P; every part's load is issued before the first is used.
// ME: compile-time bound on E.
template <int TT, int UNR, int KJMAX, int PMAX, int STRIDE = PERM_THREADS, int ME = GATE_MAX_E>
__device__ __forceinline__ void gate_partial_sums(const float* __restrict__ x,
                                                  const float* __restrict__ w_gate, int T, int d,
                                                  int E, int tid, const GatePrev& pv,
                                                  float (&ss)[GATE_NORM_MAX_T],
                                                  float (&acc)[GATE_NORM_MAX_T][ME]) {
    constexpr bool COMB = KJMAX > 0;        // KJMAX: compile-time bound on pv.k (0: no combine)
    constexpr int KJ = COMB ? KJMAX : 1;
    const bool vec = (E & 3) == 0;  // rows of w_gate are then 16-byte aligned
    for (int r0 = tid; r0 < d; r0 += UNR * STRIDE) {
        float wr[UNR][ME], xv[UNR][TT], yv[UNR][TT][KJ][PMAX];
#pragma unroll
        for (int u = 0; u < UNR; u++) {
            const int r = r0 + u * STRIDE;
#pragma unroll
            for (int e = 0; e < ME; e++) wr[u][e] = 0.f;
#pragma unroll
            for (int t = 0; t < TT; t++) {
                xv[u][t] = 0.f;
#pragma unroll
                for (int j = 0; j < KJ; j++)
#pragma unroll
                    for (int q = 0; q < PMAX; q++) yv[u][t][j][q] = 0.f;
            }
            if (r < d) {
                if (vec) {
#pragma unroll
                    for (int q = 0; q < ME / 4; q++) {
                        if (4 * q < E) {
                            const float4 v = *(const float4*)(w_gate + (size_t)r * E + 4 * q);
                            wr[u][4 * q] = v.x; wr[u][4 * q + 1] = v.y;
                            wr[u][4 * q + 2] = v.z; wr[u][4 * q + 3] = v.w;
                        }
                    }
                } else {
#pragma unroll
                    for (int e = 0; e < ME; e++)
                        if (e < E) wr[u][e] = w_gate[(size_t)r * E + e];
                }
#pragma unroll
                for (int t = 0; t < TT; t++) {
                    if (t < T) {
                        xv[u][t] = x[(size_t)t * d + r];
                        if (COMB) {
#pragma unroll
                            for (int j = 0; j < KJ; j++)
                                if (j < pv.k) {
                                    const float* p = pv.yg + (size_t)pv.pos[t * pv.k + j] * d + r;
#pragma unroll
                                    for (int q = 0; q < PMAX; q++)
                                        if (q < pv.P) yv[u][t][j][q] = p[(size_t)q * pv.pstride];
                                }
                        }
                    }
                }
            }
        }
        if (COMB) {
#pragma unroll
            for (int u = 0; u < UNR; u++) {
#pragma unroll
                for (int t = 0; t < TT; t++) {
                    if (t < T) {
                        float a = 0.f;
#pragma unroll
                        for (int j = 0; j < KJ; j++)
                            if (j < pv.k) {
                                float v = yv[u][t][j][0];  // the parts in part order
#pragma unroll
                                for (int q = 1; q < PMAX; q++)
                                    if (q < pv.P) v += yv[u][t][j][q];
                                a += pv.w[t * pv.k + j] * v;
                            }
                        xv[u][t] += a;
                    }
                }
            }
        }
#pragma unroll
        for (int u = 0; u < UNR; u++) {
#pragma unroll
            for (int t = 0; t < TT; t++) {
                ss[t] = fmaf(xv[u][t], xv[u][t], ss[t]);
#pragma unroll
                for (int e = 0; e < ME; e++) acc[t][e] = fmaf(xv[u][t], wr[u][e], acc[t][e]);
            }
        }
    }
}


template <bool NORM, int KJMAX, int PMAX>
__global__ __launch_bounds__(PERM_THREADS) void gate_small_kernel(
    const float* __restrict__ x, const float* __restrict__ w_gate, const float* __restrict__ logits_in,
    int T, int d, int E, int k, float eps, float* __restrict__ h_out, float* __restrict__ logits_out,
    int32_t* __restrict__ idx, float* __restrict__ weights, int32_t* __restrict__ counts,
    int32_t* __restrict__ offsets, int32_t* __restrict__ perm, int32_t* __restrict__ inv_perm,
    float* __restrict__ xg, const float* __restrict__ yg_prev, int n_parts_prev,
    const int32_t* __restrict__ inv_perm_prev, const float* __restrict__ weights_prev, int k_prev,
    float* __restrict__ x_out) {
    __shared__ int s_ppos[GATE_NORM_MAX_T * MOE_MAX_K];
    __shared__ float s_pw[GATE_NORM_MAX_T * MOE_MAX_K];
    __shared__ int s_cnt[MOE_MAX_E];
    __shared__ int s_off[MOE_MAX_E + 1];
    __shared__ int s_wave[PERM_WAVES * MOE_MAX_E];
    __shared__ int s_pos[GATE_MAX_T * MOE_MAX_K];
    __shared__ int s_idx[GATE_MAX_T * MOE_MAX_K];
    __shared__ float s_logits[GATE_MAX_T * GATE_MAX_E];
    __shared__ float s_inv[GATE_MAX_T];
    __shared__ float s_part[PERM_WAVES][GATE_NORM_MAX_T * (GATE_MAX_E + 1)];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    constexpr bool COMB = KJMAX > 0;
    const bool writer = (blockIdx.x == 0);
    // The partial sums read the previous block's positions and weights straight from
    // global memory (uniform addresses), so that their other loads need not wait for a
    // barrier; the LDS copies serve the row phase at the end and are published by the
    // barriers in between.
    GatePrev pv = {yg_prev, inv_perm_prev, weights_prev, k_prev, n_parts_prev,
                   (size_t)T * k_prev * d};
    if (COMB && tid < T * k_prev) {
        s_ppos[tid] = inv_perm_prev[tid];
        s_pw[tid] = weights_prev[tid];
    }

    if (NORM) {
        // T <= GATE_NORM_MAX_T here.  Per thread: rows r = tid, tid+1024, ...; partial sums
        // of x^2 and of x * w_gate[:, e] for every token, reduced over the workgroup.
        float ss[GATE_NORM_MAX_T], acc[GATE_NORM_MAX_T][GATE_MAX_E];
#pragma unroll
        for (int t = 0; t < GATE_NORM_MAX_T; t++) {
            ss[t] = 0.f;
#pragma unroll
            for (int e = 0; e < GATE_MAX_E; e++) acc[t][e] = 0.f;
        }
        // The router matrix is cold in HBM at every layer: all loads of a group of rows
        // are issued before the first use, so a thread pays the memory latency once per
        // group instead of once per row (4 rows per group for one token, else 2).
        if (T == 1)
            gate_partial_sums<1, (KJMAX * PMAX > 2 ? 2 : 4), KJMAX, PMAX>(x, w_gate, T, d, E, tid, pv, ss,
                                                                          acc);
        else
            gate_partial_sums<GATE_NORM_MAX_T, (COMB ? 1 : 2), KJMAX, PMAX>(x, w_gate, T, d, E, tid,
                                                                             pv, ss, acc);
        // wave reduce, then across the 16 waves through LDS
#pragma unroll
        for (int t = 0; t < GATE_NORM_MAX_T; t++) {
            if (t < T) {
                ss[t] = wave_sum(ss[t]);
#pragma unroll
                for (int e = 0; e < GATE_MAX_E; e++)
                    if (e < E) acc[t][e] = wave_sum(acc[t][e]);
                if (lane == 0) {
                    s_part[wave][t * (GATE_MAX_E + 1) + GATE_MAX_E] = ss[t];
#pragma unroll
                    for (int e = 0; e < GATE_MAX_E; e++)
                        if (e < E) s_part[wave][t * (GATE_MAX_E + 1) + e] = acc[t][e];
                }
            }
        }
        __syncthreads();
        if (tid < T * (GATE_MAX_E + 1)) {
            const int t = tid / (GATE_MAX_E + 1), e = tid % (GATE_MAX_E + 1);
            if (e == GATE_MAX_E || e < E) {
                float v = 0.f;
                for (int w = 0; w < PERM_WAVES; w++) v += s_part[w][t * (GATE_MAX_E + 1) + e];
                if (e == GATE_MAX_E) s_inv[t] = 1.0f / sqrtf(v / (float)d + eps);
                else s_logits[t * GATE_MAX_E + e] = v;
            }
        }
        __syncthreads();
        // logits of the normalised rows: (x . w) * inv
        if (tid < T * GATE_MAX_E) {
            const int t = tid / GATE_MAX_E, e = tid % GATE_MAX_E;
            if (e < E) {
                const float v = s_logits[tid] * s_inv[t];
                s_logits[tid] = v;
                if (writer) logits_out[(size_t)t * E + e] = v;
            }
        }
        __syncthreads();
    } else {
        if (tid < T * GATE_MAX_E) {
            const int t = tid / GATE_MAX_E, e = tid % GATE_MAX_E;
            if (e < E) s_logits[tid] = logits_in[(size_t)t * E + e];
        }
        __syncthreads();
    }

    // ---- top-k routing: 16 lanes per token (E <= 16), same contest as route_kernel ----
    {
        const int t = tid / GATE_MAX_E, gl = tid % GATE_MAX_E;
        const bool live = (t < T);
        float v = -INFINITY;
        int e = 0x7fffffff;
        if (live && gl < E) {
            v = s_logits[t * GATE_MAX_E + gl];
            e = gl;
        }
        float my_v = 0.f, top_v = 0.f;
        int my_i = 0;
        for (int j = 0; j < k; j++) {
            float bv = v;
            int be = e;
#pragma unroll
            for (int m = 1; m < GATE_MAX_E; m <<= 1) {
                const float ov = __shfl_xor(bv, m, 64);
                const int oe = __shfl_xor(be, m, 64);
                if (ov > bv || (ov == bv && oe < be)) {
                    bv = ov;
                    be = oe;
                }
            }
            if (j == 0) top_v = bv;
            if (gl == j) {
                my_v = bv;
                my_i = be;
            }
            if (e == be) {
                v = -INFINITY;
                e = 0x7fffffff;
            }
        }
        const float u = (gl < k) ? expf(my_v - top_v) : 0.f;
        float s = u;
#pragma unroll
        for (int m = 1; m < GATE_MAX_E; m <<= 1) s += __shfl_xor(s, m, 64);
        if (live && gl < k) {
            s_idx[t * k + gl] = my_i;
            if (writer) {
                idx[(size_t)t * k + gl] = my_i;
                weights[(size_t)t * k + gl] = u / s;
            }
        }
    }
    __syncthreads();

    // ---- per-expert batching on the LDS copy of idx, then the row gather ----
    const int N = T * k;
    if (N <= 64) {
        if (wave == 0) permute_indices_wave(s_idx, N, E, counts, offsets, perm, inv_perm, writer, s_pos);
    } else {
        permute_indices(s_idx, N, E, counts, offsets, perm, inv_perm, writer, s_cnt, s_off, s_wave,
                        s_pos);
    }
    __syncthreads();
    const int row_chunks = d / 4;
    // row chunk c of token t, with the pending combine + residual applied
    auto x_chunk = [&](int t, int c) -> float4 {
        float4 r = ((const float4*)(x + (size_t)t * d))[c];
        if (COMB) {
            float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
            for (int j = 0; j < k_prev; j++) {
                const float w = s_pw[t * k_prev + j];
                const float4* src = (const float4*)(yg_prev + (size_t)s_ppos[t * k_prev + j] * d) + c;
                float4 pq[PMAX];
#pragma unroll
                for (int q = 0; q < PMAX; q++)
                    if (q < n_parts_prev) pq[q] = src[(size_t)q * (pv.pstride / 4)];
                float4 v = pq[0];
#pragma unroll
                for (int q = 1; q < PMAX; q++)
                    if (q < n_parts_prev) {
                        v.x += pq[q].x; v.y += pq[q].y; v.z += pq[q].z; v.w += pq[q].w;
                    }
                a.x += w * v.x;
                a.y += w * v.y;
                a.z += w * v.z;
                a.w += w * v.w;
            }
            r.x += a.x; r.y += a.y; r.z += a.z; r.w += a.w;
        }
        return r;
    };
    for (int p = blockIdx.x; p < N; p += gridDim.x) {
        const int t = p / k;
        float4* dst = (float4*)(xg + (size_t)s_pos[p] * d);
        const float sc = NORM ? s_inv[t] : 1.0f;
        for (int c = tid; c < row_chunks; c += PERM_THREADS) {
            float4 v = x_chunk(t, c);
            if (NORM) {
                v.x *= sc; v.y *= sc; v.z *= sc; v.w *= sc;
            }
            dst[c] = v;
        }
    }
    if (NORM && writer) {
        for (int t = 0; t < T; t++) {
            const float sc = s_inv[t];
            for (int c = tid; c < row_chunks; c += PERM_THREADS) {
                float4 v = x_chunk(t, c);
                if (COMB) ((float4*)(x_out + (size_t)t * d))[c] = v;
                v.x *= sc; v.y *= sc; v.z *= sc; v.w *= sc;
                ((float4*)(h_out + (size_t)t * d))[c] = v;
            }
        }
    }
}

int moe_gate_small_launch(bool norm, const float* x, const float* w_gate, const float* logits_in,
                          int T, int d, int E, int k, float eps, float* h_out, float* logits_out,
                          int32_t* idx, float* weights, int32_t* counts, int32_t* offsets,
                          int32_t* perm, int32_t* inv_perm, float* xg, const float* yg_prev,
                          int n_parts_prev, const int32_t* inv_perm_prev, const float* weights_prev,
                          int k_prev, float* x_out, hipStream_t s) {
    const int N = T * k;
    const unsigned grid = (unsigned)(N < 32 ? N : 32);
    const bool comb = (yg_prev != nullptr);
    if (comb && !norm) return MOE_ERR_INVALID_ARG;
    if (comb && (n_parts_prev < 1 || n_parts_prev > GATE_MAX_PARTS)) return MOE_ERR_UNSUPPORTED;
#define GATE_LAUNCH(NORM, KJMAX, PMAX)                                                            \
    hipLaunchKernelGGL((gate_small_kernel<NORM, KJMAX, PMAX>), dim3(grid), dim3(PERM_THREADS), 0, \
                       s, x,                                                                      \
                       w_gate, logits_in, T, d, E, k, eps, h_out, logits_out, idx, weights,      \
                       counts, offsets, perm, inv_perm, xg, yg_prev, n_parts_prev,               \
                       inv_perm_prev, weights_prev, k_prev, x_out)
    if (comb && k_prev <= 2 && n_parts_prev == 1) GATE_LAUNCH(true, 2, 1);
    else if (comb && k_prev <= 2) GATE_LAUNCH(true, 2, GATE_MAX_PARTS);
    else if (comb && n_parts_prev == 1) GATE_LAUNCH(true, MOE_MAX_K, 1);
    else if (comb) GATE_LAUNCH(true, MOE_MAX_K, GATE_MAX_PARTS);
    else if (norm) GATE_LAUNCH(true, 0, 1);
    else GATE_LAUNCH(false, 0, 1);
#undef GATE_LAUNCH
    return moe_launch_status();
}

// ------------------------------------------------ combine + residual add ----
__global__ __launch_bounds__(256) void combine_residual_kernel(const float4* __restrict__ yg,
                                                               const int32_t* __restrict__ inv_perm,
                                                               const float* __restrict__ weights,
                                                               int T, int k, int row_chunks,
                                                               float4* __restrict__ x) {
    const int t = blockIdx.y;
    const int c = blockIdx.x * 256 + threadIdx.x;
    if (t >= T || c >= row_chunks) return;
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int j = 0; j < k; j++) {
        const float w = weights[(size_t)t * k + j];
        const float4 v = yg[(size_t)inv_perm[(size_t)t * k + j] * row_chunks + c];
        acc.x += w * v.x;
        acc.y += w * v.y;
        acc.z += w * v.z;
        acc.w += w * v.w;
    }
    float4 r = x[(size_t)t * row_chunks + c];
    r.x += acc.x; r.y += acc.y; r.z += acc.z; r.w += acc.w;
    x[(size_t)t * row_chunks + c] = r;
}

int moe_combine_residual_launch(const float* yg, const int32_t* inv_perm, const float* weights, int T,
                                int k, int d, float* x, hipStream_t s) {
    const int row_chunks = d / 4;
    dim3 grid((unsigned)((row_chunks + 255) / 256), 1);
    for (int t0 = 0; t0 < T; t0 += 65535) {
        const int tn = (T - t0) < 65535 ? (T - t0) : 65535;
        grid.y = (unsigned)tn;
        hipLaunchKernelGGL(combine_residual_kernel, grid, dim3(256), 0, s, (const float4*)yg,
                           inv_perm + (size_t)t0 * k, weights + (size_t)t0 * k, tn, k, row_chunks,
                           (float4*)(x + (size_t)t0 * d));
    }
    return moe_launch_status();
}

// ------------------------------------- combine over unsummed reduction parts ----
// The second projection of the decode kernels leaves its reduction parts as slabs
// [P][N,d]; this combine adds them in part order while it weights and gathers:
//   v      = parts[0][pos] + parts[1][pos] + ...          (pos = inv_perm[t*k+j])
//   y[t]   = (RESID ? y[t] : 0) + sum_j w[t,j] * v
// and, when asked, stores v as yg[pos] (every row of yg belongs to exactly one slot).
template <bool RESID>
__global__ __launch_bounds__(256) void combine_parts_kernel(
    const float4* __restrict__ parts, int P, size_t stride4, const int32_t* __restrict__ inv_perm,
    const float* __restrict__ weights, int T, int k, int row_chunks, float4* __restrict__ y,
    float4* __restrict__ yg_out) {
    const int t = blockIdx.y;
    const int c = blockIdx.x * 256 + threadIdx.x;
    if (t >= T || c >= row_chunks) return;
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int j = 0; j < k; j++) {
        const float w = weights[(size_t)t * k + j];
        const size_t row = (size_t)inv_perm[(size_t)t * k + j] * row_chunks + c;
        float4 v = parts[row];
        for (int p = 1; p < P; p++) {
            const float4 u = parts[(size_t)p * stride4 + row];
            v.x += u.x; v.y += u.y; v.z += u.z; v.w += u.w;
        }
        if (yg_out) yg_out[row] = v;
        acc.x += w * v.x;
        acc.y += w * v.y;
        acc.z += w * v.z;
        acc.w += w * v.w;
    }
    if (RESID) {
        float4 r = y[(size_t)t * row_chunks + c];
        r.x += acc.x; r.y += acc.y; r.z += acc.z; r.w += acc.w;
        acc = r;
    }
    y[(size_t)t * row_chunks + c] = acc;
}

int moe_combine_parts_launch(const float* parts, int n_parts, size_t part_stride,
                             const int32_t* inv_perm, const float* weights, int T, int k, int d,
                             float* y, bool residual, float* yg_out, hipStream_t s) {
    const int row_chunks = d / 4;
    dim3 grid((unsigned)((row_chunks + 255) / 256), 1);
    for (int t0 = 0; t0 < T; t0 += 65535) {
        const int tn = (T - t0) < 65535 ? (T - t0) : 65535;
        grid.y = (unsigned)tn;
        if (residual)
            hipLaunchKernelGGL(combine_parts_kernel<true>, grid, dim3(256), 0, s, (const float4*)parts,
                               n_parts, part_stride / 4, inv_perm + (size_t)t0 * k,
                               weights + (size_t)t0 * k, tn, k, row_chunks,
                               (float4*)(y + (size_t)t0 * d), (float4*)yg_out);
        else
            hipLaunchKernelGGL(combine_parts_kernel<false>, grid, dim3(256), 0, s, (const float4*)parts,
                               n_parts, part_stride / 4, inv_perm + (size_t)t0 * k,
                               weights + (size_t)t0 * k, tn, k, row_chunks,
                               (float4*)(y + (size_t)t0 * d), (float4*)yg_out);
    }
    return moe_launch_status();
}

// ------------------------------- RMSNorm + router logits for any number of tokens ----
// NL_TOK tokens per workgroup of 1024 threads, so that a row of the router matrix is loaded
// once for NL_TOK tokens; thread-strided partial sums with grouped loads (see
// gate_partial_sums), reduced over the workgroup.  NORM: h = x / rms(x) is written and
// logits = (x . w_gate) / rms(x); else logits = x . w_gate.  E <= GATE_MAX_E.
#define NL_TOK 2
#define NL_THREADS 1024
// ME: 8 or 16, bound on E (the sums of experts that do not exist cost as much as the others).
template <bool NORM, int ME>
__global__ __launch_bounds__(NL_THREADS) void norm_logits_kernel(const float* __restrict__ x,
                                                                  const float* __restrict__ w_gate,
                                                                  int T, int d, int E, float eps,
                                                                  float* __restrict__ h,
                                                                  float* __restrict__ logits,
                                                                  float* __restrict__ sums) {
    static_assert(NL_TOK <= GATE_NORM_MAX_T, "gate_partial_sums holds GATE_NORM_MAX_T tokens");
    __shared__ float s_part[NL_THREADS / 64][NL_TOK * (ME + 1)];
    __shared__ float s_inv[NL_TOK];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int t0 = blockIdx.x * NL_TOK;
    const int Tl = (T - t0) < NL_TOK ? (T - t0) : NL_TOK;
    const float* xb = x + (size_t)t0 * d;
    float ss[GATE_NORM_MAX_T], acc[GATE_NORM_MAX_T][ME];
#pragma unroll
    for (int t = 0; t < NL_TOK; t++) {
        ss[t] = 0.f;
#pragma unroll
        for (int e = 0; e < ME; e++) acc[t][e] = 0.f;
    }
    const GatePrev none = {nullptr, nullptr, nullptr, 0, 1, 0};
    gate_partial_sums<NL_TOK, 4, 0, 1, NL_THREADS, ME>(xb, w_gate, Tl, d, E, tid, none, ss, acc);
#pragma unroll
    for (int t = 0; t < NL_TOK; t++) {
        if (t < Tl) {
            ss[t] = wave_sum(ss[t]);
#pragma unroll
            for (int e = 0; e < ME; e++)
                if (e < E) acc[t][e] = wave_sum(acc[t][e]);
            if (lane == 0) {
                s_part[wave][t * (ME + 1) + ME] = ss[t];
#pragma unroll
                for (int e = 0; e < ME; e++)
                    if (e < E) s_part[wave][t * (ME + 1) + e] = acc[t][e];
            }
        }
    }
    __syncthreads();
    if (tid < Tl) {
        float v = 0.f;
        for (int w = 0; w < NL_THREADS / 64; w++) v += s_part[w][tid * (ME + 1) + ME];
        s_inv[tid] = NORM ? 1.0f / sqrtf(v / (float)d + eps) : 1.0f;
        if (NORM && sums) sums[(size_t)(t0 + tid) * (E + 1) + E] = v;  // the raw sum of squares
    }
    __syncthreads();
    if (tid < Tl * ME) {
        const int t = tid / ME, e = tid % ME;
        if (e < E) {
            float v = 0.f;
            for (int w = 0; w < NL_THREADS / 64; w++) v += s_part[w][t * (ME + 1) + e];
            if (logits) logits[(size_t)(t0 + t) * E + e] = NORM ? v * s_inv[t] : v;
            if (NORM && sums) sums[(size_t)(t0 + t) * (E + 1) + e] = v;  // the raw dot product
        }
    }
    if (NORM && h) {
        const int row_chunks = d / 4;
        for (int t = 0; t < Tl; t++) {
            const float sc = s_inv[t];
            const float4* src = (const float4*)(xb + (size_t)t * d);
            float4* dst = (float4*)(h + (size_t)(t0 + t) * d);
            for (int c = tid; c < row_chunks; c += NL_THREADS) {
                float4 v = src[c];
                v.x *= sc; v.y *= sc; v.z *= sc; v.w *= sc;
                dst[c] = v;
            }
        }
    }
}

bool moe_norm_logits_supported(int E) { return E <= GATE_MAX_E; }

// norm: h (if not null) is written too, and sums (if not null) receives the unscaled sums
// [T][E+1]: x . w_gate[:, e] at e, sum(x^2) at E; logits may then be null
int moe_norm_logits_launch(bool norm, const float* x, const float* w_gate, int T, int d, int E,
                           float eps, float* h, float* logits, float* sums, hipStream_t s) {
    const unsigned grid = (unsigned)((T + NL_TOK - 1) / NL_TOK);
#define NL_CASE(NORM, ME)                                                                                 \
    hipLaunchKernelGGL((norm_logits_kernel<NORM, ME>), dim3(grid), dim3(NL_THREADS), 0, s, x, w_gate, T, d, \
                       E, eps, h, logits, sums)
    if (norm && E <= 8) NL_CASE(true, 8);
    else if (norm) NL_CASE(true, 16);
    else if (E <= 8) NL_CASE(false, 8);
    else NL_CASE(false, 16);
#undef NL_CASE
    return moe_launch_status();
}
