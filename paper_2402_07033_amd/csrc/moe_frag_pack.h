// Per-expert bookkeeping of the routed rows (for whole waves) and the kernel that re-lays
// activations as B-operand fragments for the grouped GEMM (moe_ffn_grouped.hip).  Device code
// only.
#pragma once

#include "moe_internal.h"

// ---- segment bookkeeping: expert e owns blocks [bbase_e, bbase_e + ceil(M_e/16)) ----
struct SegInfo {
    int e;        // expert
    int row0;     // first row of the expert's segment in xg / yg
    int rows;     // rows of the segment
    int bbase;    // first packed block of the segment
};

// Expert `lane`'s rows [lo, lo + rows) of the routed rows (none for lanes >= E), for a whole
// wave.  Offsets that do not ascend or leave [0, N] are clamped as a walk over the experts
// would: lo_e = clamp(offsets[e], lo_{e-1}, N) = min(N, running max of offsets[0..e], at least
// 0); hi_e = clamp(offsets[e+1], lo_e, N).
__device__ __forceinline__ void gg_segment_of_lane(const int32_t* __restrict__ offsets, int E, int N,
                                                   int lane, int& lo, int& rows) {
    const int o0 = (lane < E) ? offsets[lane] : 0, o1 = (lane < E) ? offsets[lane + 1] : 0;
    int run = o0 < 0 ? 0 : o0;
#pragma unroll
    for (int dlt = 1; dlt < 64; dlt <<= 1) {
        const int v = __shfl_up(run, dlt, 64);
        if (lane >= dlt) run = run > v ? run : v;
    }
    lo = run > N ? N : run;
    const int hi = o1 < lo ? lo : (o1 > N ? N : o1);
    rows = hi - lo;
    if (lane >= E) {
        lo = 0;
        rows = 0;
    }
}

// Locate packed block `blk` (global block index) -> its segment; false if past the end.  For a
// whole wave: one parallel read of the offsets and two scans (a walk over the experts costs a
// memory round trip each: the pack kernel took 13 us with 64 experts, 6.5 now).
__device__ __forceinline__ bool gg_find_block(const int32_t* __restrict__ offsets, int E, int N,
                                              int blk, int lane, SegInfo& si) {
    int lo, rows;
    gg_segment_of_lane(offsets, E, N, lane, lo, rows);
    const int nb = (rows + 15) / 16;
    int inc = nb;
#pragma unroll
    for (int dlt = 1; dlt < 64; dlt <<= 1) {
        const int v = __shfl_up(inc, dlt, 64);
        if (lane >= dlt) inc += v;
    }
    const unsigned long long m = __ballot(blk >= inc - nb && blk < inc);
    if (m == 0ull) return false;
    const int e = __builtin_amdgcn_readfirstlane((int)__builtin_ctzll(m));
    si.e = e;
    si.row0 = __builtin_amdgcn_readlane(lo, e);
    si.rows = __builtin_amdgcn_readlane(rows, e);
    si.bbase = __builtin_amdgcn_readlane(inc - nb, e);
    return true;
}

// ------------------------------------------------------------------- pack ----
// blockIdx.x = packed block: rows [row0 + 16*b, +16) of a segment become d/32 B-operand
// fragments; rows past the segment end are zero.  blockIdx.y splits the block's fragments
// into ranges of GG_PACK_KS reduction steps, so that a launch with few blocks (a few hundred
// rows) still fills the chip.  With `perm` the batched row i is read as xg[perm[i] / k]: xg
// is then the token array itself and the gathered copy is never materialised.
#define GG_PACK_KS 32
template <bool ACT_BF16>
__global__ __launch_bounds__(256) void gg_pack_kernel(const void* __restrict__ xg,
                                                      const int32_t* __restrict__ perm, int k,
                                                      const int32_t* __restrict__ offsets, int E,
                                                      int N, int d, u32x4_t* __restrict__ xp) {
    SegInfo si;
    if (!gg_find_block(offsets, E, N, blockIdx.x, threadIdx.x & 63, si)) return;
    const int b = blockIdx.x - si.bbase;
    const int KS = d / 32;
    const int ks_lo = blockIdx.y * GG_PACK_KS;
    const int ks_n = (KS - ks_lo) < GG_PACK_KS ? (KS - ks_lo) : GG_PACK_KS;
    // the lane's source row is the same for every fragment of the block
    const int t = threadIdx.x & 15;
    const int r = b * 16 + t;
    int src = si.row0 + r;
    if (perm && r < si.rows) src = perm[si.row0 + r] / k;
    for (int i = threadIdx.x; i < ks_n * 64; i += 256) {
        const int lane = i & 63, ks = ks_lo + (i >> 6);
        const int kq = lane >> 4;
        u32x4_t v = {0u, 0u, 0u, 0u};
        if (r < si.rows) {
            const size_t off = (size_t)src * d + (size_t)ks * 32 + kq * 8;
            if (ACT_BF16) {
                v = *(const u32x4_t*)((const uint16_t*)xg + off);
            } else {
                const float4 v0 = *(const float4*)((const float*)xg + off);
                const float4 v1 = *(const float4*)((const float*)xg + off + 4);
                v[0] = moe_pack_bf16x2(v0.x, v0.y);
                v[1] = moe_pack_bf16x2(v0.z, v0.w);
                v[2] = moe_pack_bf16x2(v1.x, v1.y);
                v[3] = moe_pack_bf16x2(v1.z, v1.w);
            }
        }
        xp[((size_t)blockIdx.x * KS + ks) * 64 + lane] = v;
    }
}

// grid of gg_pack_kernel for `nb` packed blocks of d columns
static inline dim3 gg_pack_grid(size_t nb, int d) {
    return dim3((unsigned)nb, (unsigned)((d / 32 + GG_PACK_KS - 1) / GG_PACK_KS));
}
