// The LDS ring of the grouped GEMM's token fragments (moe_ffn_grouped.hip): how many stages it
// has, how far ahead a step requests, and the order the barriers give.  Plain constants, so
// that the order can also be replayed on the host.
//
// Step k of the loop (numbered through all tiles of a workgroup; step 0 of a tile is even)
//   1. waits until at most the requests of its last LA-1 steps are in flight,
//   2. meets the other waves at a barrier, if k is even,
//   3. requests its shares of stage k + GG_AHEAD into ring slot (k + GG_AHEAD) % NS,
//   4. multiplies with the fragments of stage k and reads those of stage k + 1; the reads are
//      waited for in step k + 1, fragment by fragment.  A tile of ten blocks has registers for
//      half a step's fragments: in step k it reads the second half of stage k and the first of
//      stage k + 1.
// So a wave's reads of stage s have returned when it ends step s, and no earlier.
#pragma once

#ifndef GG_NS
#define GG_NS 8  // LDS stages of token fragments (one KiB per token block each)
#endif
// The weight fragments of step k are requested GG_LA steps earlier into a register ring that
// is named statically, so the step loop is unrolled GG_U times (GG_LA < GG_U, reduction %
// GG_U == 0).  The depth itself matters little (2, 3, 4 and 5 steps are within 1 % at every
// size: what a CU may have in flight is full long before); the 128 x 512 tile, which requests
// twice as much per step, keeps 2 steps, because a third spills.
#ifndef GG_U
#define GG_U 4
#endif
#ifndef GG_LA
#define GG_LA 3
#endif
#ifndef GG_WIDE_LA
#define GG_WIDE_LA 2
#endif
#define GG_BARRIER_STEPS 2  // steps per barrier

// Stages requested ahead.  The slot that step k refills held stage k + GG_AHEAD - NS, which every
// wave must have finished reading before a barrier that this step is behind: with NS - 2 that is
// stage k - 2, whose reads ended in step k - 2, and step k - 1 or k has a barrier.  (With
// NS - 1 it is stage k - 1 and an odd step has no barrier between: only the latency of the
// refill would keep it behind another wave's reads.)  The depth is not what bounds the loop: with
// NS - 3 every case from 77 to 4096 tokens takes the same time within 0.4 %.
#ifndef GG_AHEAD
#define GG_AHEAD (GG_NS - 2)
#endif

// Is there a barrier step b, a multiple of GG_BARRIER_STEPS, with lo <= b <= k, for every k?
constexpr bool gg_barrier_within(int steps_back) { return steps_back + 1 >= GG_BARRIER_STEPS; }
// Refill after read: the reads of stage k + ahead - ns end with that step, so a barrier is
// needed in the steps k + ahead - ns + 1 .. k.
constexpr bool gg_refill_ordered(int ns, int ahead) { return gg_barrier_within(ns - ahead - 1); }
// Read after arrival: stage k + 1 was requested in step k + 1 - ahead and is waited for in
// step k + 1 - ahead + la; a barrier is needed from there up to step k, where it is read.
constexpr bool gg_arrival_ordered(int ahead, int la) { return gg_barrier_within(ahead - la - 1); }
