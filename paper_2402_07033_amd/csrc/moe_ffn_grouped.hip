// Prefill-sized expert FFN for gfx950: grouped GEMM on the bf16 matrix cores.
//
// Both operands of v_mfma_f32_16x16x32_bf16 are kept in fragment order (see
// moe_internal.h): the packed weights are the A operand (16 output features x
// 32 reduction indices), and the activations are first re-laid into B-operand
// fragments (32 reduction indices x 16 token rows) per expert segment, padded
// with zero rows to a multiple of 16, so that no tile straddles two experts
// and the GEMM main loop has no bounds checks.  A fragment is 1 KiB: one
// wavefront moves it with a single coalesced 16-byte-per-lane access.
//
//   pack  : xg [N,d] (fp32 or bf16) -> xp fragments [block][d/32]
//   up    : per (token tile of 256 rows, 128 h-columns): a = x.w1, b = x.w3,
//           h = silu(a)*b written as bf16 straight into B-operand fragments
//           hp [block][f/32] for the second GEMM
//   down  : per (token tile of 256 rows, 256 output features): yg = h.w2, fp32
//
// GEMM kernel (one 256 x 256 x 32 step = 1024 matrix-core clocks per SIMD).  What bounds it: a step
// takes about 0.7 us, hardly less with fewer matrix instructions.  At 4096 tokens nearly all tiles
// are full, the matrix cores are busy 72-73 % of the clocks, and the board's power holds these at
// 1.7-1.9 GHz (an earlier loop on 32x32x16 was 1.23 times as fast on all-zero tokens); at 1531 tokens,
// or with 16 experts, they are busy 55-62 % at 2.0 GHz.  Below ~200 rows per expert the weight stream bounds it
// (5.5-6.4 TB/s).
//   * workgroup tile: up to 256 token rows x 16 weight fragment rows, 4 waves, one per
//     SIMD; wave w owns fragment rows 4w..4w+3 for all token rows: 64 MFMA tiles = 256
//     accumulator registers (pinned to the accumulation register file through the inline-asm
//     constraint).  16x16x32 and not 32x32x16: in a loop of this tile's matrix instructions alone,
//     written for that comparison, the first sustained 2080 TFLOP/s on random operands, the other 1830.
//   * token rows come in units of 64 (4 blocks of 16).  An expert's units are dealt evenly to
//     its tiles, and the step loop exists once per number of units (1..4): a tile that is not
//     full issues only the matrix instructions, LDS reads and token requests of its own units.
//     Skewed routing leaves every expert's last tile partly filled: with whole tiles of 256
//     rows 34 % of the matrix work of 3062 rows (8 experts) was padding, with units 8 %.  The gain
//     in time is smaller, since a step costs the same: 16 experts, 4096 tokens, first projection
//     813 -> 771 us.
//   * weights (A) never touch LDS: each wave streams its own fragments straight from global
//     memory into a register ring, LA steps ahead (the packed layout makes these 1 KiB
//     coalesced loads with no redundancy between waves).
//   * token fragments (B) are shared by the 4 waves through a ring of NS LDS stages filled by
//     direct-to-LDS loads (no staging registers, no LDS stores); every wave reads the fragments
//     of the next step while it issues the matrix instructions of the current one (one register
//     set, refilled in place right after its last use; half a set in tiles of ten blocks, which read
//     the step's own second half, too).
//   * the requests of a step are spread between the matrix instructions, one barrier per two
//     steps publishes the next stages (the order of the ring: moe_gg_ring.h).  They are buffer loads:
//     an address is a descriptor, the lane offset and one scalar, where 64-bit pointers per request
//     filled the scalar registers (65..229 spills; 46..61 now and 94..140 in the kernels of two tile shapes, hardly
//     any of them in a step loop); 55 other instructions stand beside the
//     64 matrix instructions of a full step, 61 with pointers, one between two of them where it can be.
//   * the workgroup is persistent (one per CU) and the two load streams run across tile
//     boundaries: while the last steps of a tile are multiplied, the first stages of the next
//     one are already being requested.  The last groups of U steps of a tile are their own
//     copies of the loop body, in which it is a compile-time matter which requests belong to
//     the next tile.  The stores of a tile's result stay in flight during the next tile's first
//     steps (loads and stores share one counter, and the first step's operands are older than
//     the stores).
//   * tiles are dealt in rounds of one tile per workgroup, an XCD taking 32 neighbours of the
//     order expert, group of at most 8 token tiles, feature tile, token tile: about 8 x 4
//     tiles, which share 12 operand tiles in one L2.  Every XCD has its part of every round, so an
//     expert's size does not unbalance them; where experts of one tile and larger ones are there, they walk
//     the rounds from different starts (gg_turned in moe_gg_sched.h, with the rest of the schedule).  One contiguous range of tiles per XCD, which hits L2
//     more often, was slower: 4096 tokens 2.308 -> 2.340 ms, 1531 tokens 1.045 -> 1.056.
// Measured (kernel with whole 256-row tiles, one tile range per XCD, 64-bit pointers -> this): layer
// of 4096 tokens, 8 experts, Zipf 2.46 -> 2.35 ms; 1531 tokens 1.19 -> 1.07; 4096 tokens, 16 experts
// 1.46 -> 1.30; 77 tokens 0.518 -> 0.487; 64 experts of f = 1408, 300 tokens, k = 6 0.276 -> 0.238 (10 us of
// it the one-launch batching); a block of 512 tokens, balanced, 0.63 before and after.
#include <atomic>

#include "moe_internal.h"
#include "moe_frag_pack.h"
#include "moe_gg_ring.h"
#include "moe_gg_sched.h"

// Tile shapes (token rows x weight fragment rows of 16 features per workgroup), by the mean
// number of rows per expert:
//   256 x 16 (256 tokens x 256 features): the default;
//   192 x 16 (192 tokens x 256 features): 97..176 and 233..256 rows;
//   128 x 32 (128 tokens x 512 features): up to 96 rows -- twice the weight bytes per step,
//           which is what bounds such experts;
//   160 x 12..32 (up to 160 tokens x 192..512 features; "small experts"): in place of any of them where the offsets show
//           that no expert has more than 160 rows, and up to 96 rows wherever it fills the rounds better, decided on the device
//           (gg_small_tiles in moe_gg_sched.h).  The weight stream
//           bounds such launches.  A step moves a tile's weights W and its token rows t (mostly L2 hits) through one CU, and
//           its time follows W + t / 2 (KiB: 16 + 8 for 128 rows of the 192 x 256 tile, 32 + 8 here), until HBM is full at
//           6.5 TB/s; a round that is not full leaves bandwidth unused, so the tiles' width is cut to fill it.  First
//           projection, 8 experts of f = 14336: 8 x 128 rows 361 -> 328 us (5.2 -> 5.7 TB/s; the fix-up of its pieces, 11 us,
//           ends at once), 8 x 64 331 -> 311, 2 x 90 120 -> 97, 3 experts of 107 rows 168 -> 150; 16 of f = 6400: 16 x
//           128 349 -> 326, 16 x 40 300 -> 285, 6 x 90 158 -> 124; 64 of f = 1408: 28 rows each 134 -> 128, 24 x 24 66 -> 57.
//           With larger experts among them it is ahead up to 96 rows on average (gg_small_tiles); above, from 1 % ahead to 9
//           % behind (16 experts, 1100 tokens, Zipf 1.2 613 -> 631; second projections 179 -> 190, 199 -> 215), and not taken.
//           Ten blocks of 16 rows are 80 accumulator tiles of a wave, 64 in accumulation registers and 16 in vector
//           registers.
#define GG_THREADS 256
#define GG_SMALL_BLOCKS (GG_SMALL_ROWS / 16)  // token blocks of the small experts' tile
// The lambdas of the loop have to be inlined: as a call, with its captures in memory, the wave-uniform values
// among them become per-lane values, and every buffer request a loop over the lanes.
#define GG_INLINE __attribute__((always_inline))
// Mean rows per expert up to which the 192 x 256 tile is used (from GG_WIDE_MAX_ROWS on), and the range above it where the 256 x 256 tile comes
// first: experts of 177..232 rows on average mostly fit one 256-row tile and need two of 192.  At 36
// sizes and routings there: balanced 2-33 % ahead (200 rows: 877 -> 671 us over 8 experts, 803 -> 604
// over 16); Zipf 0.6 and 1.2, where the mean describes no expert, from 1 % behind to 8 % ahead at 23 of
// 24, 4 % behind at one (64 experts, 177 rows).  Around 250 rows half of the experts need two of either,
// and the smaller tile is 2-17 % ahead, balanced.  (In the 192-row tile's two ranges skewed routing has
// it from 11 % behind to 3 % ahead of the 256-row one, and the ranges' inner ends are not sharp:
// balanced, 172 rows 1 % ahead over 8 experts, 9 % behind over 16; 235 rows 2-12 % behind.)
#define GG_R192_MAX_ROWS 176
#define GG_R192_MIN_ROWS2 233
#define GG_R192_MAX_ROWS2 256
#define GG_GROUP 8         // token tiles that are neighbours of one weight tile, see the tile order
// 16-row token blocks per unit of a tile of NBW blocks: 4, or 2 where the tile is no multiple of 4
constexpr int gg_unit_blocks(int NBW) { return NBW % 4 == 0 ? 4 : 2; }
// Blocks of an LDS stage: each wave requests the same number.
constexpr int gg_stage_blocks(int NBW) { return (NBW + 3) / 4 * 4; }

// ------------------------------------------------------------------- GEMM ----
struct GroupedArgs {
    const u32x4_t* wfrag;  // A operand: packed weights (w13 or w2)
    const u32x4_t* bfrag;  // B operand: packed activations (xp or hp)
    const int32_t* offsets;
    void* out;  // up: hp fragments (bf16); down: yg [N,d] fp32
    int E, N;
    int KS;      // reduction steps of 32
    int FR;      // weight fragment rows per expert (up: 2*f/16, down: d/16)
    int NT;      // the launch's own tiles along the features
    int KS_out;  // up: f/32 (fragment columns of hp); down: unused
    int C;       // down: d (row length of yg)
    int split;   // gg_split_limit, or 0: nothing is cut
    float* part; // split: partial tiles [8 XCDs][workgroups per XCD][2][256*256] fp32
};

// s_waitcnt with only one counter constrained (gfx9 encoding: vmcnt = bits 3:0 and
// 15:14, expcnt = 6:4, lgkmcnt = 11:8; all-ones = no wait).
#define GG_WAIT_VMCNT(n) __builtin_amdgcn_s_waitcnt(0x0F70 | ((n) & 15) | (((n) >> 4) << 14))
#define GG_WAIT_LGKM(n) __builtin_amdgcn_s_waitcnt(0xC07F | ((n) << 8))

struct TileInfo {
    SegInfo si;
    int nt;     // feature tile
    int frow;   // its first fragment row, of the expert's
    int groups; // FLEX: groups of 4 fragment rows in it
    int blk0;   // first block of the tile inside the segment
    int nblk;   // blocks of the tile that exist
    int units;  // units of 4 blocks (the last one may hold fewer blocks)
    int once;   // the expert's only token tile: its weights are read once
    // the part of the tile's reduction this unit of work covers (whole tile: 0, KS)
    int k_lo, klen;
    bool partial;
    int piece;  // 0 or 1: which of this workgroup's two partial-tile slots it writes
};

// Logical tiles of a launch: NT * sum_e ceil(units_e / MU), in the order expert, then
// feature tile, then token tile (fastest), so that neighbouring indices share a weight tile.
// The experts' segments are decoded once per workgroup into a table in LDS
// (entry e: expert e; entries >= E hold no tiles).  A tile index is then decoded with LDS
// reads and a ballot -- no global memory access, and in particular no wait on the vector
// memory counter, which would also cover the operand loads in flight for the next tile.
#define GG_SEG_LO 0     // first row
#define GG_SEG_ROWS 1   // rows
#define GG_SEG_NB 2     // 16-row blocks
#define GG_SEG_TILES 3  // token tiles
#define GG_SEG_BASE 4   // first token tile
#define GG_SEG_BB 5     // first packed block
#define GG_SEG_FIELDS 6

// One wave fills the table (lane e: expert e), for tiles of NBW blocks; returns the number of token tiles.  SMALL:
// small = feature tiles of an expert where tiles of GG_SMALL_BLOCKS and a width of their own are taken instead (0: they are not).
template <bool UP, int NBW, int FRW, bool SMALL>
__device__ __forceinline__ int gg_seg_table(const GroupedArgs& a, int wgs, int lane, int (*tab)[64], bool write, int& small) {
    int lo, rows;
    gg_segment_of_lane(a.offsets, a.E, a.N, lane, lo, rows);
    const int nb = (rows + 15) / 16;
    small = 0;
    if (SMALL && gg_small_allowed(UP, FRW == 8, a.N, a.E, __ballot(nb > GG_SMALL_BLOCKS) != 0ull)) {
        // token tiles of 160 rows, and of the launch's own in the upper half (few: gg_small_expected)
        int t = (nb + GG_SMALL_BLOCKS - 1) / GG_SMALL_BLOCKS + ((nb + NBW - 1) / NBW << 16);
#pragma unroll
        for (int dlt = 1; dlt < 64; dlt <<= 1) t += __shfl_xor(t, dlt, 64);
        t = __builtin_amdgcn_readfirstlane(t);
        small = __builtin_amdgcn_readfirstlane(gg_small_tiles(UP, a.N, a.E, __popcll(__ballot(nb > 0)), t & 0xffff, t >> 16, a.NT,
                                                              a.FR, wgs, a.KS, a.split, FRW == 4));
    }
    const int tile_blocks = small ? GG_SMALL_BLOCKS : NBW;
    const int tiles = (nb + tile_blocks - 1) / tile_blocks;
    int inc_t = tiles, inc_b = nb;
#pragma unroll
    for (int dlt = 1; dlt < 64; dlt <<= 1) {
        const int vt = __shfl_up(inc_t, dlt, 64), vb = __shfl_up(inc_b, dlt, 64);
        if (lane >= dlt) {
            inc_t += vt;
            inc_b += vb;
        }
    }
    if (write) {
        tab[GG_SEG_LO][lane] = lo;
        tab[GG_SEG_ROWS][lane] = rows;
        tab[GG_SEG_NB][lane] = nb;
        tab[GG_SEG_TILES][lane] = tiles;
        tab[GG_SEG_BASE][lane] = inc_t - tiles;
        tab[GG_SEG_BB][lane] = inc_b - nb;
    }
    return __builtin_amdgcn_readlane(inc_t, 63);
}

// The schedule's turn, decided by one wave from the table (moe_gg_sched.h).
__device__ __forceinline__ bool gg_turned(const int (*tab)[64], int lane, int total, int NT, int KS) {
    return gg_turned(__popcll(__ballot(tab[GG_SEG_TILES][lane] == 1)), total, NT, KS);
}

// Logical tile index -> tile, from the table.  UB: blocks of a unit.
template <int UB>
__device__ __forceinline__ bool gg_decode_tile_tab(const int (*tab)[64], int lane, int NT,
                                                   int L, TileInfo& ti) {
    const int my_tiles = tab[GG_SEG_TILES][lane], my_base = tab[GG_SEG_BASE][lane] * NT;
    const unsigned long long m = __ballot(my_tiles > 0 && L >= my_base && L < my_base + my_tiles * NT);
    if (m == 0ull) return false;
    const int e = __builtin_amdgcn_readfirstlane((int)__builtin_ctzll(m));
    const int tiles = __builtin_amdgcn_readfirstlane(tab[GG_SEG_TILES][e]);
    const int nb = __builtin_amdgcn_readfirstlane(tab[GG_SEG_NB][e]);
    const int r = L - __builtin_amdgcn_readfirstlane(tab[GG_SEG_BASE][e]) * NT;
    // token tiles in groups of at most GG_GROUP, the feature tile next, the token tile fastest
    const int ng = (tiles + GG_GROUP - 1) / GG_GROUP;
    const int gq = tiles / ng, gmore = tiles % ng;  // the first gmore groups hold one tile more
    const int big = gmore * (gq + 1) * NT;
    const int gw = r < big ? gq + 1 : gq;           // width of the tile's group
    const int rr = r < big ? r : r - big;
    const int gi = rr / (gw * NT);                  // group among those of its width
    const int ro = rr - gi * (gw * NT);
    ti.nt = ro / gw;
    const int tis = (r < big ? 0 : gmore * (gq + 1)) + gi * gw + ro % gw;  // token tile inside the segment
    ti.si.e = e;
    ti.si.row0 = __builtin_amdgcn_readfirstlane(tab[GG_SEG_LO][e]);
    ti.si.rows = __builtin_amdgcn_readfirstlane(tab[GG_SEG_ROWS][e]);
    ti.si.bbase = __builtin_amdgcn_readfirstlane(tab[GG_SEG_BB][e]);
    ti.once = tiles == 1;
    // the expert's units, dealt evenly to its tiles
    const int nu = (nb + UB - 1) / UB;
    const int per = nu / tiles, more = nu % tiles;  // the first `more` tiles take one more
    ti.units = per + (tis < more ? 1 : 0);
    ti.blk0 = UB * (tis * per + (tis < more ? tis : more));
    ti.nblk = (nb - ti.blk0) < UB * ti.units ? (nb - ti.blk0) : UB * ti.units;
    ti.k_lo = 0;
    ti.klen = 0;  // filled in by the caller
    ti.partial = false;
    ti.piece = 0;
    return true;
}

// The tile's fragment rows.  FLEX: the expert's groups of 4 rows dealt evenly to its NT tiles, 3..8 for each; wave w
// holds groups w and w + 4.
template <int FRW, bool FLEX>
__device__ __forceinline__ void gg_feature_rows(int FR, int NT, TileInfo& ti) {
    if (FLEX) {
        const int groups = FR / 4, lo = ti.nt * groups / NT, hi = (ti.nt + 1) * groups / NT;
        ti.frow = lo * 4;
        ti.groups = hi - lo;
    } else {
        ti.frow = ti.nt * (4 * FRW);
        ti.groups = FRW;
    }
}
// Fragment row j of a wave inside the tile.
template <int FRW, bool FLEX>
__device__ __forceinline__ constexpr int gg_wave_row(int wave, int j) {
    return FLEX ? (j / 4) * 16 + 4 * wave + j % 4 : FRW * wave + j;
}

// Weight fragment load.  ANT: non-temporal, for a tile whose expert has no other token tile: its
// weights are read once, should not push the token fragments (re-read by every feature tile) out of
// L2, and a plain read of 1.75 GiB streams at 6.9 TB/s that way, at 6.0 otherwise.  Weights that several
// token tiles share stay in L2: past it, 27 % second tiles lose 2.5 %, 50 % lose 13 % (192-row tile).
// Chosen per tile (two more copies of the step loop for each number of units) instead of once for the
// launch by the share of second tiles, both projections: 8 experts, Zipf, 300 tokens 641 -> 627 us, 600 tokens
// 795 -> 777, 16 experts, 4096 tokens 1181 -> 1169, 64 experts, 300 tokens 224 -> 220, balanced 512 tokens 603 ->
// 599; 1531 and 4096 tokens within 0.3 %.
template <bool ANT>
__device__ __forceinline__ u32x4_t gg_ld_a(__amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff) {
    // (cache policy 2: nt)
    return __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, ANT ? 2 : 0));
}

// The lane number, recomputed where it is used and invisible to the optimiser (which would
// otherwise share it with the copy made at kernel start and keep that alive, or derive
// per-lane addresses from it ahead of the main loop).
__device__ __forceinline__ int gg_lane_opaque() {
    int l;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(l));
    return l;
}

// MFMA with the accumulator pinned to the accumulation registers: 256 of them
// are live per wave, and left to itself the register allocator shuffles them
// through the vector registers inside the loop.
__device__ __forceinline__ void gg_mfma(f32x4_t& c, const u32x4_t& a, const u32x4_t& b) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
}
// ... with a zero accumulator going in (the first step of a tile)
__device__ __forceinline__ void gg_mfma_first(f32x4_t& c, const u32x4_t& a, const u32x4_t& b) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=a"(c) : "v"(a), "v"(b));
}
// ... in vector registers: the tiles beyond the 64th of a wave
__device__ __forceinline__ void gg_mfma_v(f32x4_t& c, const u32x4_t& a, const u32x4_t& b) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(c) : "v"(a), "v"(b));
}
__device__ __forceinline__ void gg_mfma_first_v(f32x4_t& c, const u32x4_t& a, const u32x4_t& b) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=&v"(c) : "v"(a), "v"(b));
}

// Buffer descriptor over the 2 GiB of addresses from p on (p is wave-uniform, which the compiler does not
// know: without the readfirstlanes it would loop over the lanes at every use).  Operand
// requests then take one scalar add for their address: descriptor + lane offset + scalar
// offset + immediate.  An offset of GG_RSRC_BYTES is out of its range (and 16 bytes further does
// not wrap): a store there is dropped.  Offsets inside a tile stay below 1.1 GiB: 32 fragment
// rows, or 16 token blocks, of at most 32768 fragments; 256 rows of at most 2^20 floats.
#define GG_RSRC_BYTES 0x80000000u
__device__ __forceinline__ __amdgpu_buffer_rsrc_t gg_rsrc(const char* p) {
    const unsigned long long v = (unsigned long long)p;
    const unsigned lo = __builtin_amdgcn_readfirstlane((int)(unsigned)v);
    const unsigned hi = __builtin_amdgcn_readfirstlane((int)(unsigned)(v >> 32));
    return __builtin_amdgcn_make_buffer_rsrc((void*)(((unsigned long long)hi << 32) | lo), 0, (int)GG_RSRC_BYTES,
                                             0x00027000);
}

// Names the registers of ring slot u of the weight fragments where the slot is about to be used (no
// instruction).  Left to itself the register allocator gives the copies of the step loop different
// registers for fragments that are in flight from one copy to the next, and moves or spills them in
// between, which waits for them: in the 256 x 256 tile's kernels 93 (first projection) and 44 registers
// were spilled, 17 and 8 are now; 1531 tokens 1009 -> 1001 us, 4096 tokens 2257 -> 2242, both projections.
template <int I>
__device__ __forceinline__ void gg_pin(u32x4_t& x) {
    if constexpr (I == 0) asm volatile("" : "+{v[192:195]}"(x));
    else if constexpr (I == 1) asm volatile("" : "+{v[196:199]}"(x));
    else if constexpr (I == 2) asm volatile("" : "+{v[200:203]}"(x));
    else if constexpr (I == 3) asm volatile("" : "+{v[204:207]}"(x));
    else if constexpr (I == 4) asm volatile("" : "+{v[208:211]}"(x));
    else if constexpr (I == 5) asm volatile("" : "+{v[212:215]}"(x));
    else if constexpr (I == 6) asm volatile("" : "+{v[216:219]}"(x));
    else if constexpr (I == 7) asm volatile("" : "+{v[220:223]}"(x));
    else if constexpr (I == 8) asm volatile("" : "+{v[224:227]}"(x));
    else if constexpr (I == 9) asm volatile("" : "+{v[228:231]}"(x));
    else if constexpr (I == 10) asm volatile("" : "+{v[232:235]}"(x));
    else if constexpr (I == 11) asm volatile("" : "+{v[236:239]}"(x));
    else if constexpr (I == 12) asm volatile("" : "+{v[240:243]}"(x));
    else if constexpr (I == 13) asm volatile("" : "+{v[244:247]}"(x));
    else if constexpr (I == 14) asm volatile("" : "+{v[248:251]}"(x));
    else if constexpr (I == 15) asm volatile("" : "+{v[252:255]}"(x));
}
template <int SLOT>
__device__ __forceinline__ void gg_pin_slot(u32x4_t (&r)[4]) {
    gg_pin<4 * SLOT>(r[0]);
    gg_pin<4 * SLOT + 1>(r[1]);
    gg_pin<4 * SLOT + 2>(r[2]);
    gg_pin<4 * SLOT + 3>(r[3]);
}

template <int V>
struct GgInt {
    static constexpr int value = V;
};

// a / (1 + exp(-a)), to the bits of the fp32 division (16 M values of each of N(0,1), N(0,16) and
// -90..90, infinities, NaN): the reciprocal estimate, then one correction of the quotient by its
// exact residual.  The estimate is taken of a quarter of the denominator, because v_rcp_f32 flushes the
// reciprocals of denominators above 2^126 (a < -87.3) to zero.  (ldexp: 0.25 is no inline constant,
// and a register for it spills in the 256-row tile.)  The compiler's division takes 11 instructions
// where these are 8: layer of 4096 tokens 2.419 -> 2.409 ms; with the estimate alone (mean error 12 %
// larger, zero below -87.3) 2.392.
__device__ __forceinline__ float gg_silu(float a) {
    const float e = __expf(-a), den = 1.0f + e;
    const float r = __builtin_ldexpf(__builtin_amdgcn_rcpf(__builtin_ldexpf(den, -2)), -2);
    float q = a * r;
    q = __builtin_fmaf(__builtin_fmaf(-q, den, a), r, q);
    return __builtin_amdgcn_div_fixupf(q, den, a);
}

// First projection: h = silu(x.w1) * (x.w3) of two neighbouring 16-column blocks (a0, b0: the
// w1 and w3 tiles of the even block; a1, b1: of the odd one), rounded to bf16, as B fragments of
// the second GEMM.  Lane l of a tile holds token l % 16 and columns 4*(l/16) .. +3; after
// exchanging the odd 16-lane rows of the even block with the even rows of the odd block every
// lane holds eight columns, and the wave writes the token block's whole 1 KiB fragment.
__device__ __forceinline__ u32x4_t gg_make_h(const f32x4_t& a0, const f32x4_t& b0, const f32x4_t& a1,
                                             const f32x4_t& b1) {
    typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
    typedef float f2 __attribute__((ext_vector_type(2)));
    unsigned pk[4];
#pragma unroll
    for (int q = 0; q < 4; q++) {
        f2 hv;
#pragma unroll
        for (int r = 0; r < 2; r++) {
            const float av = (q < 2 ? a0 : a1)[2 * (q & 1) + r], bv = (q < 2 ? b0 : b1)[2 * (q & 1) + r];
            hv[r] = gg_silu(av) * bv;
        }
        pk[q] = __builtin_bit_cast(unsigned, __builtin_convertvector(hv, bf2));
    }
    const auto s0 = __builtin_amdgcn_permlane16_swap(pk[0], pk[2], false, false);
    const auto s1 = __builtin_amdgcn_permlane16_swap(pk[1], pk[3], false, false);
    return u32x4_t{s0[0], s1[0], s0[1], s1[1]};
}
// Byte offset of gg_make_h's value for this lane inside the fragment: lanes 16..31 and 48..63
// hold the odd column block, lanes 32..63 its columns 8..15.
__device__ __forceinline__ unsigned gg_h_off(int lane) {
    return (unsigned)(((((lane >> 4) & 1) * 2 + (lane >> 5)) * 16 + (lane & 15)) * 16);
}

// MODE: which units of work this copy of the loop covers: 0 = whole tiles and pieces, 1 = whole tiles
// only, 2 = pieces only.
// NBW x FRW: token blocks of the tile, at most, x fragment rows of a wave.
// FLEX: feature tiles of 3..8 groups of rows (gg_feature_rows); of a group that is not there a wave requests and
// stores nothing.
template <bool UP, int NBW, int FRW, bool FLEX, int MODE, int U, int LA, int NS>
__device__ __forceinline__ void gg_gemm_body(const GroupedArgs& a, int NT, int total, int split_limit, bool turned,
                                             const int (*s_seg)[64]) {
    static_assert(NBW * FRW <= 80 && NBW % 2 == 0 && FRW % 4 == 0, "at most 256 + 64 accumulators per wave");
    static_assert(LA < U && U % GG_BARRIER_STEPS == 0, "register ring; a tile starts at a barrier step");
    static_assert(gg_refill_ordered(NS, GG_AHEAD) && gg_arrival_ordered(GG_AHEAD, LA), "stage ring, see moe_gg_ring.h");
    constexpr int UB = gg_unit_blocks(NBW);
    constexpr int NSB = gg_stage_blocks(NBW);
    constexpr int NBQ = NSB / 4;       // token blocks each wave requests into LDS per step
    constexpr int TG = (GG_AHEAD + U - 1) / U;  // groups at the end of a tile that look into the next
    extern __shared__ __align__(16) unsigned char smem[];
    u32x4_t* lds = (u32x4_t*)smem;  // [NS stages][NSB fragments][64 lanes]

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // fragment rows [FRW*wave, +FRW)

    // This workgroup's units of work: whole tiles in rounds, then pieces.  When the tile count
    // is not a multiple of the workgroup count the last round would leave most CUs idle (576
    // second-projection tiles over 256 CUs = 2.25 rounds), so the left-over tiles are cut along
    // the reduction instead, in equal pieces for all workgroups; every piece stores its partial
    // sums into scratch and gg_fixup_kernel adds the pieces of a tile in a fixed order (then
    // applies SiLU*mul, first projection).
    const int xcd = blockIdx.x & 7;
    const int wgs = gridDim.x >> 3;
    const int me = blockIdx.x >> 3;
    const GgSched sc = gg_sched(total, wgs, xcd, a.KS, split_limit);
    const bool split = sc.split;
    const int last = (int)((unsigned)(me + sc.n_full) % (unsigned)wgs);  // left-over tile, if it stays whole
    const int n_full = sc.n_full + (!split && last < sc.R ? 1 : 0);
    const int turn = gg_first_round(turned, sc.n_full, xcd);
    // pieces of the left-over tiles for this workgroup
    // (plain scalars, no arrays: an array indexed at run time would live in scratch memory, and
    // every read of it would wait on the counter of the operand loads in flight)
    int pc_tile0 = 0, pc_lo0 = 0, pc_len0 = 0, pc_tile1 = 0, pc_len1 = 0, n_pieces = 0;
    if (split && sc.R > 0) {
        const int S = sc.R * a.KS;
        const int c0 = gg_piece_cut(me, S, a.KS, wgs, U, NS), c1 = gg_piece_cut(me + 1, S, a.KS, wgs, U, NS);
        if (c0 < c1) {
            const int rA = c0 / a.KS;
            const int endA = c1 < (rA + 1) * a.KS ? c1 : (rA + 1) * a.KS;
            pc_tile0 = rA; pc_lo0 = c0 - rA * a.KS; pc_len0 = endA - c0;
            n_pieces = 1;
            if (c1 > endA) {
                pc_tile1 = rA + 1; pc_len1 = c1 - endA;  // starts at step 0 of its tile
                n_pieces = 2;
            }
        }
    }
    // uniform values, pinned to scalar registers (the compiler otherwise keeps them in a table
    // in scratch memory for the selection below)
    pc_tile0 = __builtin_amdgcn_readfirstlane(pc_tile0);
    pc_lo0 = __builtin_amdgcn_readfirstlane(pc_lo0);
    pc_len0 = __builtin_amdgcn_readfirstlane(pc_len0);
    pc_tile1 = __builtin_amdgcn_readfirstlane(pc_tile1);
    pc_len1 = __builtin_amdgcn_readfirstlane(pc_len1);
    n_pieces = __builtin_amdgcn_readfirstlane(n_pieces);
    const int n_units = (MODE == 1) ? n_full : n_full + n_pieces;
    auto unit_at = [&](int n, TileInfo& ti) GG_INLINE -> bool {
        if (n >= n_units) return false;
        int L, lo = 0, len = a.KS;
        if (n < n_full) {
            const int r = n + turn;
            L = n < sc.n_full ? gg_round_slot(r < sc.n_full ? r : r - sc.n_full, wgs, xcd, me) : sc.left_lo + last;
        } else {
            // first or second piece, selected by arithmetic (a two-way choice on n is turned
            // into a table in scratch memory by the compiler)
            const int first = (n == n_full) ? 1 : 0;
            L = sc.left_lo + pc_tile1 + first * (pc_tile0 - pc_tile1);
            lo = first * pc_lo0;
            len = pc_len1 + first * (pc_len0 - pc_len1);
        }
        // (the lane number is recomputed here, opaquely, so that no address derived from it
        // has to stay in a register through the main loop; see the epilogue)
        const int lane_d = gg_lane_opaque();
        if (!gg_decode_tile_tab<UB>(s_seg, lane_d, NT, L, ti)) return false;
        gg_feature_rows<FRW, FLEX>(a.FR, NT, ti);
        ti.k_lo = lo;
        ti.klen = len;
        ti.partial = (n >= n_full);  // pieces always go through scratch and the fix-up
        ti.piece = n < n_full ? 0 : n - n_full;
        return true;
    };

    // Operand addresses: the tile's base, a scalar offset that walks along the reduction (1 KiB
    // per step) and the lane's 16 bytes of the fragment.  A: row j of this wave.  B: block 4v + wave
    // of the tile is request v of this wave; blocks past the tile's last one repeat it (every wave always has its requests, their products are never stored).  (Offsets
    // inside a tile: at most 32 rows of f/32 <= 32768 fragments, 1 GiB.)
    const unsigned row_bytes = (unsigned)a.KS * 1024u;  // one fragment row / token block
    const unsigned voff = (unsigned)lane * 16u;
    // the lane's offset of a weight request: behind the descriptor, which returns zeros without a memory access,
    // for a group of rows that the tile does not have
    auto has = [&](const TileInfo& ti, int j) GG_INLINE -> bool { return !FLEX || wave + (j / 4) * 4 < ti.groups; };
    auto a_voff = [&](const TileInfo& ti, int j) GG_INLINE -> unsigned { return has(ti, j) ? voff : GG_RSRC_BYTES; };
    auto a_row = [&](int j) GG_INLINE -> unsigned { return (unsigned)gg_wave_row<FRW, FLEX>(0, j) * row_bytes; };
    auto a_base = [&](const TileInfo& ti) GG_INLINE -> const char* {
        return (const char*)a.wfrag +
               (((size_t)ti.si.e * a.FR + (size_t)ti.frow + gg_wave_row<FRW, FLEX>(wave, 0)) * a.KS + ti.k_lo) * 1024;
    };
    auto b_base = [&](const TileInfo& ti) GG_INLINE -> const char* {
        return (const char*)a.bfrag + ((size_t)(ti.si.bbase + ti.blk0) * a.KS + ti.k_lo) * 1024;
    };
    auto b_off = [&](const TileInfo& ti, unsigned (&vo)[NBQ]) GG_INLINE {
#pragma unroll
        for (int v = 0; v < NBQ; v++) {
            const int blk = 4 * v + wave;
            vo[v] = __builtin_amdgcn_readfirstlane((unsigned)(blk < ti.nblk ? blk : ti.nblk - 1) * row_bytes);
        }
    };
    // request v of this wave for stage number `gstage`, `soff` bytes along the reduction
    auto issue_b = [&](__amdgpu_buffer_rsrc_t r, unsigned soff, unsigned gstage, int v) GG_INLINE {
        unsigned char* dst = smem + ((gstage % NS) * (NSB * 1024) + wave * 1024);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(
            r, (__attribute__((address_space(3))) void*)(dst + v * 4096), 16, voff, soff, 0, 0);
    };

    int unit = (MODE == 2) ? n_full : 0;
    TileInfo cur, nxt;
    if (!unit_at(unit, cur)) return;
    nxt = cur;
    bool has_next = unit_at(unit + 1, nxt);
    if (!has_next) nxt = cur;  // behind the last unit: its own first steps again, never used
    const char *pa = a_base(cur), *pb = b_base(cur);
    const char *pa_n = a_base(nxt), *pb_n = b_base(nxt);
    unsigned vo_b[NBQ], vo_bn[NBQ];
    b_off(cur, vo_b);
    b_off(nxt, vo_bn);
    constexpr int GR = FLEX ? FRW / 4 : 1;
    unsigned va[GR], va_n[GR];
#pragma unroll
    for (int q = 0; q < GR; q++) {
        va[q] = a_voff(cur, 4 * q);
        va_n[q] = a_voff(nxt, 4 * q);
    }

    u32x4_t areg[U][FRW];  // [ring slot][fragment row]

    // ---- prologue of the first tile: request stages 0..GG_AHEAD-1 and A of steps 0..LA-1 ----
    {
        const __amdgpu_buffer_rsrc_t ra = gg_rsrc(pa), rb = gg_rsrc(pb);
        for (int j = 0; j < GG_AHEAD; j++)
#pragma unroll
            for (int v = 0; v < NBQ; v++) issue_b(rb, vo_b[v] + j * 1024, j, v);
#pragma unroll
        for (int s = 0; s < LA; s++)
#pragma unroll
            for (int j = 0; j < FRW; j++) areg[s][j] = gg_ld_a<false>(ra, va[j / 4 % GR], s * 1024 + a_row(j));
    }
    GG_WAIT_VMCNT(0);
    __builtin_amdgcn_s_barrier();

    unsigned g = 0;  // running step count of this workgroup: LDS stage g % NS

    int stores = 0;  // store instructions of the previous tile's epilogue (at least)

    // one tile of B token blocks (B = 4 * units)
    // (its last groups request the next tile's first weights, with this tile's policy)
    auto tile = [&](auto blocks, auto once) GG_INLINE {
        constexpr int B = decltype(blocks)::value;
        constexpr bool ANT = decltype(once)::value != 0;
        constexpr int NBB = (B + 3) / 4;
        constexpr int VMIN = FRW + NBB;  // requests of a step, at least
        // token fragments in registers: a whole step's, or a ring of half as many where the accumulators
        // need the registers
        constexpr int RB = B * FRW > 64 ? B / 2 : B;
        f32x4_t acc[B][FRW];
        u32x4_t breg[RB];
        g = __builtin_amdgcn_readfirstlane(g);
        const __amdgpu_buffer_rsrc_t ra = gg_rsrc(pa), rb = gg_rsrc(pb), ra_n = gg_rsrc(pa_n), rb_n = gg_rsrc(pb_n);
        unsigned kb = 0;  // bytes along the reduction: 1024 * step of the group's first step
        const int klen = __builtin_amdgcn_readfirstlane(cur.klen);
        {
            const u32x4_t* pl = lds + (g % NS) * NSB * 64 + lane;
#pragma unroll
            for (int i = 0; i < RB; i++) breg[i] = pl[i * 64];
        }
        GG_WAIT_LGKM(0);

        // U steps.  Q: how many groups are left in the tile, this one included, or 0: more than
        // TG.  A request for step u + look-ahead of the group lies in the next tile when that is
        // beyond the Q groups.  FIRST: the tile's first group.
        auto group = [&](auto left, auto first) GG_INLINE {
            constexpr int Q = decltype(left)::value;
            constexpr bool FIRST = decltype(first)::value != 0;
            constexpr int NB = Q ? NBQ : NBB;  // token requests per step (the next tile may need all)
            constexpr int VREQ = FRW + NB;
#pragma unroll
            for (int u = 0; u < U; u++) {
                // The weights of step k were requested LA steps ago, after that step's requests
                // for stage k+GG_AHEAD-LA; requests retire in order, so with at most the last
                // LA-1 steps' worth still in flight they have arrived, and so have the stages
                // requested before them (at least up to stage k+2).  (Steps issue VMIN
                // requests or more.)  In a tile's first LA steps the previous tile's stores lie
                // between those requests and the younger ones and may stay in flight as well.
                __builtin_amdgcn_sched_barrier(0);
                if (FIRST && u < LA) {
                    constexpr int V0 = (LA - 1) * VMIN;
                    if (stores >= 32) GG_WAIT_VMCNT(V0 + 32 < 63 ? V0 + 32 : 63);
                    else if (stores >= 16) GG_WAIT_VMCNT(V0 + 16);
                    else if (stores >= 8) GG_WAIT_VMCNT(V0 + 8);
                    else GG_WAIT_VMCNT(V0);
                } else {
                    GG_WAIT_VMCNT((LA - 1) * VMIN);
                }
                if constexpr (NBW == 16) {
                    static_assert(U == 4 && FRW == 4, "four slots of four fragments");
                    if (u == 0) gg_pin_slot<0>(areg[0]);
                    else if (u == 1) gg_pin_slot<1>(areg[1]);
                    else if (u == 2) gg_pin_slot<2>(areg[2]);
                    else gg_pin_slot<3>(areg[3]);
                }
                // One barrier per TWO steps: at an even step every wave has waited for its
                // shares of stages k+1 and k+2 (see above), so both are published here; and the
                // slots refilled during steps k and k+1 held stages k-2 and k-1, whose reads
                // every wave has waited for in its steps k-2 and k-1.
                if (u % GG_BARRIER_STEPS == 0) __builtin_amdgcn_s_barrier();
                const u32x4_t* pc = lds + ((g + u) % NS) * NSB * 64 + lane;
                const u32x4_t* pl = lds + ((g + u + 1) % NS) * NSB * 64 + lane;
                auto refill = [&](const int i) GG_INLINE {  // the fragment RB blocks behind block i
                    breg[i % RB] = i + RB < B ? pc[(i + RB) * 64] : pl[(i + RB - B) * 64];
                };
                auto issue = [&](const int v) GG_INLINE {
                    if (v < NB) {
                        const int jb = u + GG_AHEAD;  // step of the group
                        if (Q == 0 || jb < Q * U)
                            issue_b(rb, vo_b[v] + kb + jb * 1024, g + jb, v);
                        else
                            issue_b(rb_n, vo_bn[v] + (jb - Q * U) * 1024, g + jb, v);
                    } else {
                        const int ja = u + LA, j = v - NB;
                        if (Q == 0 || ja < Q * U)
                            areg[ja % U][j] = gg_ld_a<ANT>(ra, va[j / 4 % GR], kb + ja * 1024 + a_row(j));
                        else
                            areg[ja % U][j] = gg_ld_a<ANT>(ra_n, va_n[j / 4 % GR], (ja - Q * U) * 1024 + a_row(j));
                    }
                };
                // One other instruction at most between two matrix instructions where it can be: a
                // matrix instruction takes 16 clocks and the wave issues one instruction per 4, so
                // runs of others (they stood behind every eighth, seven in a row) leave the
                // matrix cores idle.  The order over the tile is a snake: from one matrix instruction to the
                // next only one of the two operands changes, which costs less power, and power bounds
                // the clock of full tiles.  (Masks: scalar instructions may move.)  Runs and no snake ->
                // this, both projections: 4096 tokens Zipf 2187 -> 2130 us, 8 x 1024 rows 2036 -> 1978, 1531
                // tokens Zipf 995 -> 972; about half of it each.
#pragma unroll
                for (int i = 0; i < B; i++) {
                    // LDS reads return in order: with at most that many younger ones in flight,
                    // the fragments of blocks i and i + 1 have arrived
                    if (i == 0) GG_WAIT_LGKM(RB - 2);
                    else if ((i & 1) == 0) GG_WAIT_LGKM(RB - 3);
#pragma unroll
                    for (int jj = 0; jj < FRW; jj++) {
                        const int j = (i & 1) ? FRW - 1 - jj : jj;
                        __builtin_amdgcn_sched_barrier(4);
                        if (i * FRW < 64) {
                            if (FIRST && u == 0) gg_mfma_first(acc[i][j], areg[u][j], breg[i % RB]);
                            else gg_mfma(acc[i][j], areg[u][j], breg[i % RB]);
                        } else {
                            if (FIRST && u == 0) gg_mfma_first_v(acc[i][j], areg[u][j], breg[i % RB]);
                            else gg_mfma_v(acc[i][j], areg[u][j], breg[i % RB]);
                        }
                        __builtin_amdgcn_sched_barrier(4);
                        if (jj == 0 && i > 0) refill(i - 1);
                        // the vector-memory requests are spread evenly over the blocks, so that the
                        // requests of the four waves never queue up in front of the matrix
                        // instructions
#pragma unroll
                        for (int v = 0; v < VREQ; v++)
                            if ((((2 * v + 1) * B * FRW / (2 * VREQ)) & ~3) + 2 == i * FRW + jj) issue(v);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
                refill(B - 1);
            }
            g += U;
            kb += U * 1024;
        };
        int k = klen - TG * U;
        if (k > 0) {
            group(GgInt<0>{}, GgInt<1>{});
            for (k -= U; k > 0; k -= U) group(GgInt<0>{}, GgInt<0>{});
            if constexpr (TG >= 2) group(GgInt<2>{}, GgInt<0>{});
        } else {
            if constexpr (TG >= 2) group(GgInt<2>{}, GgInt<1>{});
        }
        group(GgInt<1>{}, GgInt<0>{});
        static_assert(TG == 2, "tail groups");

        // ---- epilogue of the tile (the next tile's loads are in flight) ----
        // the compiler cannot see the MFMAs: cover the matrix-core write -> read hazard
        asm volatile("s_nop 15\n s_nop 15" ::: "memory");
        // The epilogue's per-lane addresses are derived from a copy of the lane number that the
        // compiler cannot trace back to the one above: it would otherwise compute them before
        // the main loop and keep them in registers through it.
        const int lane_e = gg_lane_opaque();
        const int t = lane_e & 15;  // token in block
        // Every store is issued, so that their number is known (see the waits above): those of
        // rows, blocks or features that do not exist lie beyond the descriptor and are dropped.
        if (MODE == 2 || (MODE == 0 && cur.partial)) {
            // piece of a tile: raw partial sums to this workgroup's slot, in the order of the
            // accumulators (whole lines); the fix-up kernel adds the pieces
            const __amdgpu_buffer_rsrc_t rs = gg_rsrc(
                (const char*)(a.part + (((size_t)xcd * wgs + me) * 2 + cur.piece) * (256 * 256) + wave * (NBW * FRW * 256)));
#pragma unroll
            for (int i = 0; i < B; i++) {
                const unsigned vo = i < cur.nblk ? (unsigned)lane_e * 16u : GG_RSRC_BYTES;
#pragma unroll
                for (int j = 0; j < FRW; j++)
                    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, acc[i][j]), rs, vo,
                                                           (i * FRW + j) * 1024, 0);
            }
            stores = B * FRW;
        } else if (UP) {
            // fragment rows 4jj..4jj+3 of this wave: w1, w3 of an even and of the next column block
            const int ks_o = (cur.frow + gg_wave_row<FRW, FLEX>(wave, 0)) / 4;  // h fragment column of jj = 0
            const __amdgpu_buffer_rsrc_t rs = gg_rsrc(
                (const char*)a.out + ((size_t)(cur.si.bbase + cur.blk0) * a.KS_out + ks_o) * 1024);
            const unsigned vo = gg_h_off(lane_e);
#pragma unroll
            for (int i = 0; i < B; i++)
#pragma unroll
                for (int jj = 0; jj < FRW / 4; jj++) {
                    const u32x4_t hv = gg_make_h(acc[i][4 * jj], acc[i][4 * jj + 1], acc[i][4 * jj + 2],
                                                 acc[i][4 * jj + 3]);
                    const unsigned o = vo + (unsigned)i * (unsigned)a.KS_out * 1024u + gg_wave_row<FRW, FLEX>(0, 4 * jj) * 256u;
                    __builtin_amdgcn_raw_buffer_store_b128(hv, rs, i < cur.nblk && has(cur, 4 * jj) ? o : GG_RSRC_BYTES, 0, 0);
                }
            stores = B * (FRW / 4);
        } else {
            const int r0 = cur.blk0 * 16;  // first row of the tile inside the segment
            const __amdgpu_buffer_rsrc_t rs = gg_rsrc(
                (const char*)((float*)a.out + (size_t)(cur.si.row0 + r0) * a.C + (cur.frow + gg_wave_row<FRW, FLEX>(wave, 0)) * 16));
            const int rows = cur.si.rows - r0;
            const unsigned vo = (unsigned)t * (unsigned)a.C * 4u + (unsigned)(lane_e >> 4) * 16u;
#pragma unroll
            for (int i = 0; i < B; i++)
#pragma unroll
                for (int j = 0; j < FRW; j++) {
                    const unsigned o = i * 16 + t < rows && has(cur, j) ? vo + (unsigned)(i * 16) * (unsigned)a.C * 4u
                                                                        : GG_RSRC_BYTES;
                    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, acc[i][j]), rs,
                                                           o + gg_wave_row<FRW, FLEX>(0, j) * 64, 0, 0);
                }
            stores = B * FRW;
        }
    };

    for (;;) {
        // by the number of units of the tile, 1 .. NBW / 4
        auto units = [&](auto once) GG_INLINE {
            if (NBW == 10) {
                if (cur.units <= 2) tile(GgInt<4>{}, once);
                else if (cur.units == 3) tile(GgInt<6>{}, once);
                else if (cur.units == 4) tile(GgInt<8>{}, once);
                else tile(GgInt<NBW == 10 ? 10 : 8>{}, once);
            } else if (cur.units == 1) tile(GgInt<4>{}, once);
            else if (NBW == 8 || cur.units == 2) tile(GgInt<8>{}, once);
            else if constexpr (NBW >= 12) {
                if (NBW == 12 || cur.units == 3) tile(GgInt<12>{}, once);
                else if constexpr (NBW >= 16) tile(GgInt<16>{}, once);
            }
        };
        if (cur.once) units(GgInt<1>{});
        else units(GgInt<0>{});
        if (!has_next) {
            // the unconditional look-ahead of the last steps is still in flight (some of it on
            // its way into LDS): it must land before the workgroup gives its LDS back
            GG_WAIT_VMCNT(0);
            break;
        }
        // advance: next becomes current; look one unit further ahead
        unit++;
        cur = nxt;
        pa = pa_n;
        pb = pb_n;
#pragma unroll
        for (int v = 0; v < NBQ; v++) vo_b[v] = vo_bn[v];
        has_next = unit_at(unit + 1, nxt);
        if (!has_next) nxt = cur;
        pa_n = a_base(nxt);
        pb_n = b_base(nxt);
        b_off(nxt, vo_bn);
#pragma unroll
        for (int q = 0; q < GR; q++) {
            va[q] = va_n[q];
            va_n[q] = a_voff(nxt, 4 * q);
        }
        GG_WAIT_LGKM(0);  // the decode's reads must not sit in the LDS read counter
    }
}

// The first projection's whole tiles and pieces are two copies of the loop, one after the other: an
// epilogue with both the SiLU body and the raw store spills 153-289 registers in the 8 x 8 and 16 x 4 tiles.
template <bool UP, int NBW, int FRW, bool SMALL, int U, int LA, int NS>
__global__ __launch_bounds__(GG_THREADS) void gg_gemm_kernel(GroupedArgs a) {
    __shared__ int s_seg[GG_SEG_FIELDS][64];
    int small;
    const int n_tok = gg_seg_table<UP, NBW, FRW, SMALL>(a, (int)(gridDim.x >> 3), threadIdx.x & 63, s_seg, threadIdx.x < 64, small);
    __syncthreads();
    const int NT = SMALL && small ? small : a.NT, total = n_tok * NT;
    const bool turned = gg_turned(s_seg, threadIdx.x & 63, total, NT, a.KS);
    if (SMALL && small) {  // whole tiles only
        gg_gemm_body<UP, GG_SMALL_BLOCKS, 8, true, 1, GG_U, GG_WIDE_LA, GG_NS>(a, NT, total, 0, turned, s_seg);
        return;
    }
    gg_gemm_body<UP, NBW, FRW, false, UP ? 1 : 0, U, LA, NS>(a, NT, total, a.split, turned, s_seg);
    if (UP) {
        __syncthreads();  // no wave fills the LDS ring anew while another still reads it
        gg_gemm_body<UP, NBW, FRW, false, 2, U, LA, NS>(a, NT, total, a.split, turned, s_seg);
    }
}

// Adds the pieces of every left-over tile in the order of the workgroups that produced them
// (deterministic), then does what the GEMM's epilogue does for a whole tile.  Item = (left-over
// tile, token block); thread = (wave, lane) of the GEMM.  The grid is of a fixed size (the host
// does not know the number of tiles) and walks the items; every wave finds the pieces of a tile
// for itself, from the cut points the GEMM workgroups used.  Loads of two pieces are in flight
// together: one piece at a time, with a workgroup per item of the largest possible number of
// tiles, took 40 us instead of 17 for the second projection at 8192 rows.
#define GG_FIX_GRID 1024
template <bool UP, int NBW, int FRW, bool SMALL>
__global__ __launch_bounds__(256) void gg_fixup_kernel(GroupedArgs a, int wgs, int unit, int ns) {
    constexpr int FROWS = 4 * FRW;
    // the segment table as in the GEMM: one parallel read of the offsets and two wave scans
    // instead of a walk over the experts with one memory round trip each
    __shared__ int s_seg[GG_SEG_FIELDS][64];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int small;
    const int total = gg_seg_table<UP, NBW, FRW, SMALL>(a, wgs, lane, s_seg, threadIdx.x < 64, small) * a.NT;
    const int left = total % (wgs * 8);
    if (small || left == 0 || !gg_sched(total, wgs, 0, a.KS, a.split).split) return;
    __syncthreads();
    for (int item = blockIdx.x; item < left * NBW; item += gridDim.x) {
        // (tile fastest: neighbouring workgroups, and not the same ones again, take blocks that exist)
        const int lt = item % left, i = item / left;
        // XCD whose left-over tiles hold tile lt (their ranges are cut as in gg_sched)
        int xcd = (int)((unsigned)lt * 8u / (unsigned)left);
        while (left * (xcd + 1) / 8 <= lt) xcd++;
        while (left * xcd / 8 > lt) xcd--;
        const GgSched sc = gg_sched(total, wgs, xcd, a.KS, a.split);
        const int r = sc.n_full * wgs * 8 + lt - sc.left_lo;  // tile number among the XCD's
        TileInfo ti;
        if (!gg_decode_tile_tab<gg_unit_blocks(NBW)>(s_seg, lane, a.NT, sc.left_lo + r, ti)) return;
        if (i >= ti.nblk) continue;
        // lane w looks at workgroup w's cut: it holds at most one piece of this tile; a ballot
        // keeps the pieces in workgroup order (wgs <= 64)
        const int S = sc.R * a.KS;
        int slot = -1;
        if (lane < wgs) {
            const int c0 = gg_piece_cut(lane, S, a.KS, wgs, unit, ns),
                      c1 = gg_piece_cut(lane + 1, S, a.KS, wgs, unit, ns);
            if (c0 < c1) {
                const int rA = c0 / a.KS;
                const int endA = c1 < (rA + 1) * a.KS ? c1 : (rA + 1) * a.KS;
                if (rA == r) slot = (xcd * wgs + lane) * 2 + 0;
                else if (c1 > endA && rA + 1 == r) slot = (xcd * wgs + lane) * 2 + 1;
            }
        }
        unsigned long long m = __ballot(slot >= 0);
        f32x4_t c[FRW];
#pragma unroll
        for (int j = 0; j < FRW; j++) c[j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        const float* src = a.part + (size_t)(wave * NBW + i) * (FRW * 256) + lane * 4;
        while (m) {
            const float* p0 = src + (size_t)__builtin_amdgcn_readlane(slot, (int)__builtin_ctzll(m)) * (256 * 256);
            m &= m - 1;
            const bool two = m != 0ull;
            const float* p1 = two ? src + (size_t)__builtin_amdgcn_readlane(slot, (int)__builtin_ctzll(m)) * (256 * 256) : p0;
            m &= m - 1;
            f32x4_t v0[FRW], v1[FRW];
#pragma unroll
            for (int j = 0; j < FRW; j++) v0[j] = *(const f32x4_t*)(p0 + j * 256);
#pragma unroll
            for (int j = 0; j < FRW; j++) v1[j] = *(const f32x4_t*)(p1 + j * 256);
#pragma unroll
            for (int j = 0; j < FRW; j++) {
                c[j] += v0[j];
                if (two) c[j] += v1[j];
            }
        }
        const int blk = ti.blk0 + i;  // block inside the segment
        if (UP) {
            const int ks_o = ti.nt * (FROWS / 4) + (FRW / 4) * wave;
            unsigned char* dst = (unsigned char*)a.out + ((size_t)(ti.si.bbase + blk) * a.KS_out + ks_o) * 1024 +
                                 gg_h_off(lane);
#pragma unroll
            for (int jj = 0; jj < FRW / 4; jj++)
                *(u32x4_t*)(dst + jj * 1024) = gg_make_h(c[4 * jj], c[4 * jj + 1], c[4 * jj + 2], c[4 * jj + 3]);
        } else {
            const int row = blk * 16 + (lane & 15);
            if (row < ti.si.rows) {
                float* dst = (float*)a.out + (size_t)(ti.si.row0 + row) * a.C + (ti.nt * FROWS + FRW * wave) * 16 +
                             4 * (lane >> 4);
#pragma unroll
                for (int j = 0; j < FRW; j++) *(f32x4_t*)(dst + j * 16) = c[j];
            }
        }
    }
}

// ---------------------------------------------------------------- host side ----
// Kernel variants by rows per expert (see the tile shapes at the top of the file): token
// blocks and fragment rows of the tile, unroll / weight look-ahead / LDS stages of the loop.
// (_S: kernels that hold the small experts' tile as well.)
enum GgVariant { GG_STD = 0, GG_WIDE = 1, GG_R192 = 2, GG_STD_S = 3, GG_WIDE_S = 4, GG_R192_S = 5, GG_NVARIANTS = 6 };
struct GgShape { int tb, frows, u, la, ns; };
static size_t gg_lds_bytes(const GgShape& sh) {
    const int nb = gg_stage_blocks(sh.tb), small = gg_stage_blocks(GG_SMALL_BLOCKS);
    return (size_t)sh.ns * (nb > small ? nb : small) * MOE_FRAG_BYTES;
}
static GgShape gg_shape(GgVariant v) {
    switch (v) {
        case GG_WIDE:
        case GG_WIDE_S: return {8, 32, GG_U, GG_WIDE_LA, GG_NS};
        case GG_R192:
        case GG_R192_S: return {12, 16, GG_U, GG_LA, GG_NS};
        default: return {16, 16, GG_U, GG_LA, GG_NS};
    }
}

template <bool UP>
const void* gg_kernel_ptr(GgVariant v) {
    switch (v) {
        case GG_WIDE: return (const void*)gg_gemm_kernel<UP, 8, 8, false, GG_U, GG_WIDE_LA, GG_NS>;
        case GG_WIDE_S: return (const void*)gg_gemm_kernel<UP, 8, 8, true, GG_U, GG_WIDE_LA, GG_NS>;
        case GG_R192: return (const void*)gg_gemm_kernel<UP, 12, 4, false, GG_U, GG_LA, GG_NS>;
        case GG_R192_S: return (const void*)gg_gemm_kernel<UP, 12, 4, true, GG_U, GG_LA, GG_NS>;
        case GG_STD_S: return (const void*)gg_gemm_kernel<UP, 16, 4, true, GG_U, GG_LA, GG_NS>;
        default: return (const void*)gg_gemm_kernel<UP, 16, 4, false, GG_U, GG_LA, GG_NS>;
    }
}

// One projection: the persistent GEMM and the fix-up of the pieces.
template <bool UP>
int gg_launch_projection(GroupedArgs& a, GgVariant v, unsigned pgrid, hipStream_t s) {
    const GgShape sh = gg_shape(v);
    const int wgs = (int)(pgrid / 8);
    void* params[1] = {(void*)&a};
    const size_t lds_bytes = gg_lds_bytes(sh);
    MOE_HIP_TRY(hipLaunchKernel(gg_kernel_ptr<UP>(v), dim3(pgrid), dim3(GG_THREADS), params, lds_bytes, s));
    if (a.split) {
        const dim3 fgrid(GG_FIX_GRID);
#define GG_FIXUP(NBW, FRW, SMALL) \
    hipLaunchKernelGGL((gg_fixup_kernel<UP, NBW, FRW, SMALL>), fgrid, dim3(256), 0, s, a, wgs, sh.u, sh.ns)
        switch (v) {
            case GG_WIDE: GG_FIXUP(8, 8, false); break;
            case GG_WIDE_S: GG_FIXUP(8, 8, true); break;
            case GG_R192: GG_FIXUP(12, 4, false); break;
            case GG_R192_S: GG_FIXUP(12, 4, true); break;
            case GG_STD_S: GG_FIXUP(16, 4, true); break;
            default: GG_FIXUP(16, 4, false);
        }
#undef GG_FIXUP
    }
    return MOE_OK;
}

// The second projection's kernels are compiled in a file of their own, beside the first's (a minute and a half each).
#ifdef GG_SECOND_PROJECTION
template const void* gg_kernel_ptr<false>(GgVariant);
template int gg_launch_projection<false>(GroupedArgs&, GgVariant, unsigned, hipStream_t);
#else
extern template const void* gg_kernel_ptr<false>(GgVariant);
extern template int gg_launch_projection<false>(GroupedArgs&, GgVariant, unsigned, hipStream_t);

static inline size_t gg_align256(size_t v) { return (v + 255) & ~(size_t)255; }
static inline size_t gg_max_blocks(int N, int E) { return (size_t)N / 16 + E; }

// scratch for the partial tiles of the second projection: 2 slots of 256 x 256 fp32 per
// persistent workgroup (one workgroup per CU, rounded up to a multiple of 8)
static inline size_t gg_part_bytes() {
    return (size_t)((moe_num_cus() + 7) / 8 * 8) * 2 * 256 * 256 * sizeof(float);
}

size_t moe_ffn_grouped_workspace(int N, int E, int d, int f) {
    const size_t nb = gg_max_blocks(N, E);
    return gg_align256(nb * 16 * d * 2) + gg_align256(nb * 16 * f * 2) + gg_part_bytes();
}

// Second projection with fewer reduction steps than the pipelined kernel's stages (f = 128, which
// MID serves): one wave per (token block, fragment row), straight from the fragments.
#define GG_SHORT_FEATURES 64
__global__ __launch_bounds__(256) void gg_down_short_kernel(GroupedArgs a) {
    SegInfo si;
    const int lane = threadIdx.x & 63;
    if (!gg_find_block(a.offsets, a.E, a.N, blockIdx.x, lane, si)) return;
    const int fr = blockIdx.y * 4 + (threadIdx.x >> 6);  // FR is a multiple of 4
    const u32x4_t* w = a.wfrag + ((size_t)si.e * a.FR + fr) * a.KS * 64 + lane;
    const u32x4_t* h = a.bfrag + (size_t)blockIdx.x * a.KS * 64 + lane;
    f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
    for (int ks = 0; ks < a.KS; ks++)
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, w[ks * 64]),
                                                      __builtin_bit_cast(bf16x8_t, h[ks * 64]), acc, 0, 0, 0);
    const int row = ((int)blockIdx.x - si.bbase) * 16 + (lane & 15);
    if (row < si.rows)
        *(f32x4_t*)((float*)a.out + (size_t)(si.row0 + row) * a.C + fr * 16 + 4 * (lane >> 4)) = acc;
}

// The step loop is unrolled u times and the ring holds ns stages.
static bool gg_fits(GgVariant v, int ks) {
    const GgShape sh = gg_shape(v);
    return ks % sh.u == 0 && ks >= sh.ns;
}

// What a projection of variant v is launched with.
struct GgProjection {
    GgVariant v;  // with the tile of 160 rows, too, or not
    int NT, split;
};
// least: experts in use, at least (if there are fewer all the same, only the time depends on it).
static GgProjection gg_projection(GgVariant v, bool up, int N, int E, int FR, int KS, int least) {
    const GgShape sh = gg_shape(v);
    const int wgs = (moe_num_cus() + 7) / 8;
    GgProjection p = {v, FR / sh.frows, gg_split_limit(up, KS, wgs)};
    if (!gg_small_expected(up, v == GG_WIDE, N, E, FR, KS, wgs)) return p;
    p.v = v == GG_WIDE ? GG_WIDE_S : v == GG_R192 ? GG_R192_S : GG_STD_S;
    if (up && N <= GG_WIDE_MAX_ROWS * E && !gg_up_may_cut(N, E, least, 16 * sh.tb, p.NT, FR, KS, wgs, v != GG_WIDE)) p.split = 0;
    return p;
}

// Variant of each projection by the mean number of rows per expert (the host never sees the
// real counts): up to GG_WIDE_MAX_ROWS the 128-token x 512-feature tile (needs f % 256 == 0
// for the first projection, d % 512 == 0 for the second; each falls back on its own), then the
// 192-token x 256-feature one in its two ranges, else 256 x 256.
// short_down: the second projection's reduction is too short for the pipelined kernel (f = 128).
static bool gg_choose(int N, int E, int d, int f, GgVariant& vu, GgVariant& vd, bool& short_down) {
    // up tile = 16 fragment rows = 8 column blocks x (w1,w3): f % 128 == 0;
    // down tile = 256 features: d % 256 == 0; both give reductions of >= 8 steps, step
    // counts that are multiples of 4.
    if (f % 128 != 0 || d % 256 != 0) return false;
    const long long mean_rows = ((long long)N + E - 1) / E;
    vu = vd = GG_STD;
    if (mean_rows <= GG_WIDE_MAX_ROWS) {
        if (f % 256 == 0) vu = GG_WIDE;
        if (d % 512 == 0) vd = GG_WIDE;
    } else if (mean_rows <= GG_R192_MAX_ROWS ||
               (mean_rows >= GG_R192_MIN_ROWS2 && mean_rows <= GG_R192_MAX_ROWS2)) {
        vu = vd = GG_R192;
    }
    // a variant whose loop does not fit a reduction gives way to the standard one
    if (!gg_fits(vu, d / 32)) vu = GG_STD;
    if (!gg_fits(vd, f / 32)) vd = GG_STD;
    short_down = !gg_fits(vd, f / 32);
    return gg_fits(vu, d / 32);
}

// GROUPED refuses f = 128, MID serves it up to a number of rows of its own (a forced path beyond
// it stays refused); everything else is the same for both.
static bool gg_path_choose(bool mid, int N, int E, int d, int f, GgVariant& vu, GgVariant& vd, bool& short_down) {
    if (mid && (size_t)N / 192 + E > 192) return false;
    return gg_choose(N, E, d, f, vu, vd, short_down) && (mid || !short_down);
}

int moe_ffn_grouped_plan(bool mid, int N, int E, int d, int f, moe_ffn_plan_t* plan) {
    GgVariant vu, vd;
    bool short_down;
    if (!gg_path_choose(mid, N, E, d, f, vu, vd, short_down)) return MOE_ERR_UNSUPPORTED;
    const GgShape su = gg_shape(vu), sd = gg_shape(vd);
    plan->up_tile_rows = 16 * su.tb;
    plan->up_tile_features = 16 * su.frows;
    plan->down_tile_rows = short_down ? 16 : 16 * sd.tb;
    plan->down_tile_features = short_down ? GG_SHORT_FEATURES : 16 * sd.frows;
    return MOE_OK;
}

// The tiles of one projection for these rows per expert, by the functions that the kernels themselves go by.
static moe_ffn_tiles_t gg_tiles(const GgProjection& p, bool up, const int32_t* counts, int N, int E, int FR, int KS) {
    const GgShape sh = gg_shape(p.v);
    const int wgs = (moe_num_cus() + 7) / 8;
    const bool wide = sh.frows == 32;
    int active = 0, small_tok = 0, own_tok = 0, most = 0, small = 0;
    for (int e = 0; e < E; e++) {
        active += counts[e] > 0;
        small_tok += (counts[e] + GG_SMALL_ROWS - 1) / GG_SMALL_ROWS;
        own_tok += (counts[e] + 16 * sh.tb - 1) / (16 * sh.tb);
        most = counts[e] > most ? counts[e] : most;
    }
    if (p.v >= GG_STD_S && gg_small_allowed(up, wide, N, E, most > GG_SMALL_ROWS))
        small = gg_small_tiles(up, N, E, active, small_tok, own_tok, p.NT, FR, wgs, KS, p.split, !wide);
    moe_ffn_tiles_t t = {};
    t.rows = small ? GG_SMALL_ROWS : 16 * sh.tb;
    t.feature_tiles = small ? small : p.NT;
    t.features = small ? (FR / 4 + small - 1) / small * 64 : 16 * sh.frows;
    t.tiles = (small ? small_tok : own_tok) * t.feature_tiles;
    t.pieces = !small && t.tiles % (8 * wgs) && gg_sched(t.tiles, wgs, 0, KS, p.split).split;
    t.fixup = p.split != 0;
    return t;
}

int moe_ffn_grouped_tiles(bool mid, const int32_t* counts, int N, int E, int d, int f, int k, moe_ffn_tiles_t* up,
                          moe_ffn_tiles_t* down) {
    GgVariant vu, vd;
    bool short_down;
    if (!gg_path_choose(mid, N, E, d, f, vu, vd, short_down)) return MOE_ERR_UNSUPPORTED;
    const int fu = f / 8, fd = d / 16;  // fragment rows per expert
    *up = gg_tiles(gg_projection(vu, true, N, E, fu, d / 32, k < E ? k : E), true, counts, N, E, fu, d / 32);
    if (!short_down) {
        *down = gg_tiles(gg_projection(vd, false, N, E, fd, f / 32, 0), false, counts, N, E, fd, f / 32);
        return MOE_OK;
    }
    *down = {16, GG_SHORT_FEATURES, d / GG_SHORT_FEATURES, 0, 0, 0};
    for (int e = 0; e < E; e++) down->tiles += (counts[e] + 15) / 16 * down->feature_tiles;
    return MOE_OK;
}

static int gg_launch(const moe_weights* W, const void* xg, moe_dtype_t act_dtype, const int32_t* perm,
                     int k, const int32_t* offsets, int N, void* ws, float* yg, GgVariant vu, GgVariant vd,
                     bool short_down, hipStream_t s) {
    const int d = W->d, f = W->f, E = W->E;
    const size_t nb = gg_max_blocks(N, E);
    u32x4_t* xp = (u32x4_t*)ws;
    u32x4_t* hp = (u32x4_t*)((unsigned char*)ws + gg_align256(nb * 16 * d * 2));
    const unsigned pgrid = (unsigned)((moe_num_cus() + 7) / 8 * 8);  // persistent: one per CU

    // once per device; threads that race here set the same attributes
    static std::atomic<int> attr_set[MOE_MAX_DEVICES];
    const int dev = moe_current_device();
    if (dev < 0) return MOE_ERR_HIP;
    if (!attr_set[dev].load(std::memory_order_acquire)) {
        for (int v = 0; v < GG_NVARIANTS; v++) {
            const GgShape sh = gg_shape((GgVariant)v);
            const void* all[2] = {gg_kernel_ptr<true>((GgVariant)v), gg_kernel_ptr<false>((GgVariant)v)};
            for (int i = 0; i < 2; i++)
                MOE_HIP_TRY(hipFuncSetAttribute(all[i], hipFuncAttributeMaxDynamicSharedMemorySize,
                                                (int)gg_lds_bytes(sh)));
        }
        attr_set[dev].store(1, std::memory_order_release);
    }

    if (act_dtype == MOE_BF16)
        hipLaunchKernelGGL(gg_pack_kernel<true>, gg_pack_grid(nb, d), dim3(256), 0, s, xg, perm, k,
                           offsets, E, N, d, xp);
    else
        hipLaunchKernelGGL(gg_pack_kernel<false>, gg_pack_grid(nb, d), dim3(256), 0, s, xg, perm, k,
                           offsets, E, N, d, xp);

    // scratch of the pieces of left-over tiles, behind the two fragment buffers
    float* part = (float*)((unsigned char*)ws + gg_align256(nb * 16 * d * 2) +
                           gg_align256(nb * 16 * f * 2));

    const GgProjection pu = gg_projection(vu, true, N, E, f / 8, d / 32, k < E ? k : E);

    GroupedArgs up;
    up.wfrag = (const u32x4_t*)W->w13;
    up.bfrag = xp;
    up.offsets = offsets;
    up.out = hp;
    up.E = E; up.N = N;
    up.KS = d / 32;
    up.FR = 2 * (f / 16);
    up.NT = pu.NT;
    up.split = pu.split;
    up.KS_out = f / 32;
    up.C = 0;
    up.part = part;
    int rc = gg_launch_projection<true>(up, pu.v, pgrid, s);
    if (rc != MOE_OK) return rc;
    moe_record_mid_event(s);

    GroupedArgs dn;
    dn.wfrag = (const u32x4_t*)W->w2;
    dn.bfrag = hp;
    dn.offsets = offsets;
    dn.out = yg;
    dn.E = E; dn.N = N;
    dn.KS = f / 32;
    dn.FR = d / 16;
    dn.KS_out = 0;
    dn.C = d;
    dn.part = part;
    if (short_down) {
        hipLaunchKernelGGL(gg_down_short_kernel, dim3((unsigned)nb, (unsigned)(d / GG_SHORT_FEATURES)), dim3(256), 0, s, dn);
        return moe_launch_status();
    }
    const GgProjection pd = gg_projection(vd, false, N, E, d / 16, f / 32, 0);
    dn.NT = pd.NT;
    dn.split = pd.split;
    rc = gg_launch_projection<false>(dn, pd.v, pgrid, s);
    if (rc != MOE_OK) return rc;
    return moe_launch_status();
}

// MID had kernels of its own (a wave streamed two adjacent fragment rows for up to 192 rows); with
// token units the grouped GEMM's tiles are ahead at every size.  Up to 96 rows per expert (128 x 512
// tile): 8 experts, 60..380 tokens, balanced 494..575 -> 468..551 us, Zipf 505..792 -> 464..680; 64
// experts of f = 1408, 200..1000 tokens 268..489 -> 188..297.  Above, the tiles of GROUPED: 8 experts,
// 480..800 tokens, balanced 650..1117 -> 575..671, Zipf 939..1119 -> 739..851 (the 128 x 512 tile there,
// too: 660..773, slower than what it replaced up to 175 rows per expert).
int moe_ffn_grouped_launch(bool mid, const moe_weights* W, const void* xg, moe_dtype_t act_dtype,
                           const int32_t* perm, int k, const int32_t* offsets, int N, void* ws,
                           float* yg, hipStream_t s) {
    GgVariant vu, vd;
    bool short_down;
    if (!gg_path_choose(mid, N, W->E, W->d, W->f, vu, vd, short_down)) return MOE_ERR_UNSUPPORTED;
    return gg_launch(W, xg, act_dtype, perm, k, offsets, N, ws, yg, vu, vd, short_down, s);
}

bool moe_ffn_grouped_supported(bool mid, int N, int E, int d, int f) {
    GgVariant vu, vd;
    bool short_down;
    return gg_path_choose(mid, N, E, d, f, vu, vd, short_down);
}
#endif  // GG_SECOND_PROJECTION
