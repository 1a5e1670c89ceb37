// fp32 expert FFN (fp32 weights and activations, fp32 products and sums): the exact-dtype path of
// the tiny all-fp32 workload, on v_mfma_f32_16x16x4_f32.
//
// At that size (a handful of rows per expert, reductions of a few hundred) latency bounds it: what
// counts is how many dependent memory round trips a launch makes.  A workgroup of 8 waves takes
// (up to 16*RT*NT rows of one expert) x (16*FT output features); its waves split the reduction and,
// for NT > 1, the row tiles (RT of 16 rows each per wave), and request everything they need of up to 64 reduction indices at once; the
// waves' sums meet in LDS and are added in wave order.  Measured at 16 tokens, d = 256, f = 512, 8
// experts: 6.0 + 4.6 us (LDS-staged steps of 16 reduction indices, a memory round trip and two
// barriers each, and a walk over the experts before them, took 29 + 40 us); the layer of 128
// tokens, d = 512, f = 1024 223 -> 53 us.
#include "moe_internal.h"
#include "moe_frag_pack.h"

#define F32_WAVES 8
#define F32_GROUP 16  // reduction indices per group: lane quarter q takes 4q .. 4q+3
#define F32_BATCH 4   // groups requested together

// Row tile `tile` of the per-expert segments -> (expert, first row, row count), for a whole wave.
__device__ __forceinline__ bool f32_find_tile(const int32_t* __restrict__ offsets, int E, int N,
                                              int tile, int TR, int lane, int& e_out, int& row0,
                                              int& rows) {
    int lo, n;
    gg_segment_of_lane(offsets, E, N, lane, lo, n);
    const int tiles = (n + TR - 1) / TR;
    int inc = tiles;
#pragma unroll
    for (int dlt = 1; dlt < 64; dlt <<= 1) {
        const int v = __shfl_up(inc, dlt, 64);
        if (lane >= dlt) inc += v;
    }
    const unsigned long long m = __ballot(tile >= inc - tiles && tile < inc);
    if (m == 0ull) return false;
    const int e = __builtin_amdgcn_readfirstlane((int)__builtin_ctzll(m));
    const int first = tile - __builtin_amdgcn_readlane(inc - tiles, e);  // tile inside the segment
    const int left = __builtin_amdgcn_readlane(n, e) - first * TR;
    e_out = e;
    row0 = __builtin_amdgcn_readlane(lo, e) + first * TR;
    rows = left < TR ? left : TR;
    return true;
}

// UP:   out[i,c] = silu(sum_r act[i,r] wA[e,r,c]) * (sum_r act[i,r] wB[e,r,c])
// !UP:  out[i,c] = sum_r act[i,r] wA[e,r,c]
// Lane l of a matrix instruction: row tile row l % 16, features c0 + FT*(l % 16) + 0..FT-1 (one
// load of FT floats serves FT instructions), reduction indices 4*(l / 16) + s in instruction s.
template <bool UP, int FT, int NT, int RT>
__global__ __launch_bounds__(64 * F32_WAVES) void ffn_f32_kernel(
    const float* __restrict__ act, const int32_t* __restrict__ perm, int perm_k,
    const float* __restrict__ wA, const float* __restrict__ wB, const int32_t* __restrict__ offsets,
    int E, int N, int K, int C, float* __restrict__ out) {
    constexpr int NM = UP ? 2 : 1;
    constexpr int KW = F32_WAVES / NT;  // waves that share one row tile's reduction
    typedef float fvec __attribute__((ext_vector_type(FT)));
    __shared__ f32x4_t s_sum[F32_WAVES][NM][FT][RT][64];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int e, row0, rows;
    if (!f32_find_tile(offsets, E, N, blockIdx.y, 16 * RT * NT, lane, e, row0, rows)) return;
    const int nt = wave % NT, kw = wave / NT;
    const int t = lane & 15, q = lane >> 4;
    const int c0 = blockIdx.x * 16 * FT;
    // this lane's rows; rows past the end read the tile's first row and are not stored
    const float* xr[RT];
#pragma unroll
    for (int j = 0; j < RT; j++) {
        const int r = (nt * RT + j) * 16 + t;
        int src = row0 + (r < rows ? r : 0);
        if (perm) src = perm[src] / perm_k;
        xr[j] = act + (size_t)src * K + 4 * q;
    }
    const float* w[NM];
    w[0] = wA + (size_t)e * K * C + (size_t)(4 * q) * C + c0 + FT * t;
    if (UP) w[NM - 1] = wB + (size_t)e * K * C + (size_t)(4 * q) * C + c0 + FT * t;
    f32x4_t acc[NM][FT][RT];
#pragma unroll
    for (int m = 0; m < NM; m++)
#pragma unroll
        for (int i = 0; i < FT; i++)
#pragma unroll
            for (int j = 0; j < RT; j++) acc[m][i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    const int groups = K / F32_GROUP;
    if (nt * RT * 16 < rows) {
        for (int g0 = kw; g0 < groups; g0 += KW * F32_BATCH) {
            f32x4_t xv[F32_BATCH][RT];
            fvec wv[F32_BATCH][NM][4];
#pragma unroll
            for (int b = 0; b < F32_BATCH; b++) {
                // (a group past the end of the reduction: the batch's first one again, not used)
                const size_t k0 = (size_t)(g0 + b * KW < groups ? g0 + b * KW : g0) * F32_GROUP;
#pragma unroll
                for (int j = 0; j < RT; j++) xv[b][j] = *(const f32x4_t*)(xr[j] + k0);
#pragma unroll
                for (int m = 0; m < NM; m++)
#pragma unroll
                    for (int s = 0; s < 4; s++) wv[b][m][s] = *(const fvec*)(w[m] + (k0 + s) * C);
            }
            // all of the batch's loads are issued before the first is used (left to itself the
            // compiler keeps to few registers and waits several times)
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int b = 0; b < F32_BATCH; b++) {
                if (g0 + b * KW >= groups) continue;
#pragma unroll
                for (int s = 0; s < 4; s++)
#pragma unroll
                    for (int m = 0; m < NM; m++)
#pragma unroll
                        for (int i = 0; i < FT; i++)
#pragma unroll
                            for (int j = 0; j < RT; j++)
                                acc[m][i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                                    wv[b][m][s][i], xv[b][j][s], acc[m][i][j], 0, 0, 0);
            }
        }
    }
#pragma unroll
    for (int m = 0; m < NM; m++)
#pragma unroll
        for (int i = 0; i < FT; i++)
#pragma unroll
        for (int j = 0; j < RT; j++) s_sum[wave][m][i][j][lane] = acc[m][i][j];
    __syncthreads();
    // wave `wave` finishes the tiles (row tile, i) number wave, wave + 8, ...
    for (int item = wave; item < NT * RT * FT; item += F32_WAVES) {
        const int it = item / FT, i = item % FT;
        f32x4_t sum[NM];
#pragma unroll
        for (int m = 0; m < NM; m++) {
            sum[m] = s_sum[it / RT][m][i][it % RT][lane];
#pragma unroll
            for (int k2 = 1; k2 < KW; k2++) sum[m] += s_sum[k2 * NT + it / RT][m][i][it % RT][lane];
        }
        const int row = it * 16 + t;
        if (row >= rows) continue;
        // lane l holds instruction rows 4q .. 4q+3, i.e. features c0 + FT*(4q + r) + i
        float* dst = out + (size_t)(row0 + row) * C + c0 + FT * 4 * q + i;
#pragma unroll
        for (int rr = 0; rr < 4; rr++) {
            float v = sum[0][rr];
            if (UP) v = v / (1.0f + expf(-v)) * sum[NM - 1][rr];
            dst[FT * rr] = v;
        }
    }
}

size_t moe_ffn_f32_workspace(int N, int E, int d, int f) {
    (void)E;
    (void)d;
    return (size_t)N * f * sizeof(float);
}

template <bool UP>
static void ffn_f32_projection(const float* act, const int32_t* perm, int perm_k, const float* wA,
                               const float* wB, const int32_t* offsets, int E, int N, int K, int C,
                               float* out, hipStream_t s) {
    // rows per workgroup by the mean number of rows per expert: more of them share a read of the
    // weights; fewer leave more waves to a reduction.  (4096 tokens, d = 1024, f = 3584: 2.98 ms with
    // 128 rows, 3.80 with 64, 3.70 with the LDS-staged 32 x 64 tile that this replaces.)
    const int mean = (N + E - 1) / E;
    const int nt = mean <= 16 ? 1 : (mean <= 32 ? 2 : 4);
    const int rt = mean <= 64 ? 1 : 2;
    const unsigned tiles = (unsigned)(N / (16 * nt * rt) + E);  // >= sum_e ceil(M_e / rows of a tile)
    // 32 features per workgroup (whole 128-byte lines of the weight rows) unless that leaves CUs
    // without a workgroup
    const int ft = (long long)(C / 32) * tiles >= moe_num_cus() ? 2 : 1;
#define F32_CASE(FT, NT, RT)                                                                           \
    if (ft == FT && nt == NT && rt == RT)                                                              \
        hipLaunchKernelGGL((ffn_f32_kernel<UP, FT, NT, RT>), dim3((unsigned)(C / (16 * FT)), tiles),  \
                           dim3(64 * F32_WAVES), 0, s, act, perm, perm_k, wA, wB, offsets, E, N, K, C, \
                           out);
    F32_CASE(1, 1, 1)
    F32_CASE(1, 2, 1)
    F32_CASE(1, 4, 1)
    F32_CASE(2, 1, 1)
    F32_CASE(2, 2, 1)
    F32_CASE(2, 4, 1)
    F32_CASE(1, 4, 2)
    F32_CASE(2, 4, 2)
#undef F32_CASE
}

// the largest call served (gridDim.y)
bool moe_ffn_f32_supported(int N, int E) { return N / 32 + E <= 65535; }

int moe_ffn_f32_launch(const moe_weights* W, const float* xg, const int32_t* perm, int k,
                       const int32_t* offsets, int N, void* ws, float* yg, hipStream_t s) {
    if (!moe_ffn_f32_supported(N, W->E)) return MOE_ERR_UNSUPPORTED;
    float* h = (float*)ws;
    ffn_f32_projection<true>(xg, perm, k, (const float*)W->w1f, (const float*)W->w3f, offsets, W->E, N,
                             W->d, W->f, h, s);
    moe_record_mid_event(s);
    ffn_f32_projection<false>((const float*)h, (const int32_t*)nullptr, 1, (const float*)W->w2f,
                              (const float*)nullptr, offsets, W->E, N, W->f, W->d, yg, s);
    return moe_launch_status();
}
