// How the grouped GEMM (moe_ffn_grouped.hip) deals its tiles to its workgroups: rounds of whole
// tiles, the tiles of the last, incomplete round, and where these are cut.  Plain functions, so
// that the schedule can also be replayed on the host.
//
// Tiles are numbered 0 .. total-1 (expert, group of token tiles, feature tile, token tile); 8 * wgs
// workgroups, wgs for each XCD.
#pragma once

#ifndef GG_WIDE_MAX_ROWS
#define GG_WIDE_MAX_ROWS 96  // mean rows per expert up to which the 128 x 512 tile is used
#endif
#define GG_SMALL_ROWS 160    // rows of the small experts' tile
// Fragments (KiB) of a projection's weights from which the small experts' tile is considered: smaller ones stay in the
// last-level cache from call to call, and then a tile's own matrix instructions bound it (all ten blocks of 8 rows of a wave, however
// narrow the tile): 8 experts of d = 512, f = 1024, skewed 52 -> 61 us, of 1024, 2304 74 -> 79 (balanced 67 -> 63); 4 of 2048, 8192 (268
// MB) 116..134 -> 99..112.
#define GG_SMALL_MIN_FRAGS (128 << 10)

// (inlined always: what a called function returns is no wave-uniform value)
#define GG_FN constexpr __attribute__((always_inline)) inline

// Whole tiles go out in n_full rounds of one tile per workgroup.  The tiles of the last, incomplete
// round are dealt to the XCDs evenly, and cut there along the reduction so that all workgroups
// take part -- or left whole, one for each of the first workgroups: pieces store and
// re-read their partial sums, work at different steps of tiles that would otherwise share operands in L2, and a
// round that is nearly full saves little; with few workgroups at work the others' power goes to them.  Measured,
// pieces (fix-up included) -> whole:
//   first projection, 128 steps, 3..7 rounds before: 0.06..0.38 of a round 355..683 -> 401..695 us, 0.69 462 -> 482,
//     0.75..0.97 294 -> 292 (77 tokens), 440 -> 433, 386 -> 331; 8..15 rounds before, 20 sizes and routings: 0.01..0.2
//     790..1172 -> 832..1206 (0.3..5 %), 0.25..0.4 0.3..3 % (4096 tokens 1441 -> 1446), 0.5 even, 0.59 749 -> 759 and
//     792 -> 788, 0.75 887 -> 864; 25 and 56 rounds even; 64 steps: 0.04..0.08 443..456 ->
//     458..468, 0.46 267 -> 271, 0.75 140 -> 135;
//   second projection: 448 steps, 0.19..0.5 of a round 146..209 -> 281..351, 0.62 279 -> 288 and 328 -> 332, 0.69 313 -> 296,
//     0.75 402 -> 335, 0.88 469 -> 347; 200 steps: 0.5 258 -> 287, 0.69 427 -> 437, 0.75 449 -> 450, 460 -> 435; 8 rounds
//     before and 0.06..0.25 of one: 448 steps 2560..2618 -> 2763..2773, 200 steps 1282..1318 -> 1341..1351, 128 steps
//     893 -> 918.
#define GG_SPLIT_UP 22          // 32nds of a round up to which the first projection's left-over tiles are cut
#define GG_SPLIT_DOWN 20        // the second's
#define GG_SPLIT_MIN_STEPS 36   // steps that cutting has to save (of what it saves at best)
#define GG_SPLIT_KS 64          // steps of the reduction from which tiles are cut
// Left-over tiles are cut if they are at most this many 32nds of a round (0: never).  Pieces of >= 32 steps
// go to scratch and a fix-up kernel adds them; it lists the pieces of a tile with one wave, hence at
// most 64 workgroups per XCD.
GG_FN int gg_split_limit(bool up, int KS, int wgs) {
    return KS >= GG_SPLIT_KS && wgs <= 64 ? (up ? GG_SPLIT_UP : GG_SPLIT_DOWN) : 0;
}
struct GgSched {
    int n_full;   // rounds of whole tiles
    int left_lo;  // this XCD's left-over tiles: [left_lo, left_lo + R)
    int R;
    bool split;   // are they cut in pieces
};
GG_FN GgSched gg_sched(int total, int wgs, int xcd, int KS, int split) {
    GgSched sc{};
    const int W = wgs * 8;
    sc.n_full = total / W;
    const int left = total - sc.n_full * W;
    const int lo = left * xcd / 8, hi = left * (xcd + 1) / 8;
    sc.left_lo = sc.n_full * W + lo;
    sc.R = hi - lo;
    sc.split = left * 32 <= W * split && (W - left) * KS >= W * GG_SPLIT_MIN_STEPS;
    return sc;
}
// Feature tiles per expert for n_tok token tiles of up to 160 rows (N rows in all) and 3 .. 8 groups of 4 fragment
// rows, all left whole: the fewest where they fill their rounds, else as many as the rounds hold, which are narrower, of 3
// groups and more.  0: the launch's own tiles, where cutting those of the last round is better (split: gg_split_limit).  Pieces of 160
// x 512 themselves cost more to add up: second projection of 8 x 128 rows 176 + 17 us, 180 + 12 with pieces of 192 x 256; of
// 8 x 150 198 + 20, 193 + 13.  only_wide: 0 for 4 groups as well, as the launch's own tiles have: these keep more requests
// in flight (16 x 128 rows 169 -> 159).  Otherwise these have 512 features, too, and with few rows nearly full rounds of them fill
// HBM as they are: 77 tokens 460 -> 462 narrowed, 4 x 24 rows 140 -> 143 (0.88 of a round), 64 experts of f = 1408, second projection
// 55 -> 55 (0.78), 62 -> 64 (0.9), 58 -> 63 (0.73); 8 x 64 331 -> 311, 4 x 90 151 -> 147.  gg_flex_fill: without these
// questions.
// Narrowed -> cut, GEMM and fix-up: one round, 0.44 of it filled by the fewest tiles, 128 steps 87 -> 101 us, 97 -> 125
// (24, 90 rows per expert); 0.59 111 -> 134, 124 -> 160; 0.5, 200 steps 142 -> 155; 0.41 129 -> 138, 140 -> 164; 0.34 123 ->
// 120, 141 -> 146.  Two rounds, 128 steps: 1.09 of them filled 194 -> 200, 229 -> 208; 1.27 236 -> 233, 265 -> 252; 1.31 234 ->
// 231, 265 -> 256; 1.37 264 -> 256; 1.46 250 -> 260, 283 -> 295; 1.53 269 -> 272, 299 -> 301; 1.56 285 -> 300, 326 -> 349;
// 64 steps, 1.17 108 -> 115, 124 -> 130.  Narrowed -> whole and not full: 1.75 298 -> 304, 311 -> 331; 0.88 143 -> 139
// (HBM is full either way), 147 -> 151.
#define GG_FLEX_FEW_ROWS 32
#define GG_FLEX_CUT_STEPS1 120  // steps that the idle part of the round is worth, one round
#define GG_FLEX_CUT_STEPS 75    // ... several
GG_FN int gg_flex_fill(int n_tok, int groups, int wgs) {
    const int least = (groups + 7) / 8, W = wgs * 8, total = n_tok * least;
    if (n_tok == 0) return least;
    const int fill = (total + W - 1) / W * W / n_tok, most = fill < groups / 3 ? fill : groups / 3;
    return most > least ? most : least;
}
GG_FN int gg_flex(int N, int n_tok, int groups, int wgs, int KS, int split, bool only_wide) {
    const int least = (groups + 7) / 8, W = wgs * 8, total = n_tok * least;
    const int slots = (total + W - 1) / W * W;
    if (n_tok == 0 || (!only_wide && N <= GG_FLEX_FEW_ROWS * n_tok && (slots - total) * 10 <= 3 * W)) return 0;
    const int NT = gg_flex_fill(n_tok, groups, wgs);
    if (total < slots && gg_sched(total, wgs, 0, KS, split).split &&
        ((slots - total) * KS >= W * (slots == W ? GG_FLEX_CUT_STEPS1 : GG_FLEX_CUT_STEPS) || NT * n_tok * 4 < slots * 3 ||
         NT == least))
        return 0;
    return only_wide && groups <= 4 * NT ? 0 : NT;
}
// The same for the first projection up to GG_WIDE_MAX_ROWS rows per expert, where experts of more than 160 rows do not rule
// these tiles out: always, but for a few cases, most of them of few experts in use.
// Where the tiles leave 48 steps' worth of the one round idle, cutting is better: a step takes 0.47 us however narrow its tile
// is.  GEMM, narrowed -> cut, fix-up and 1.2 us between them included, 128 steps: 1 expert of f = 6400, 16..128 rows, 60..76 -> 39..50
// us, 2 of them 66 -> 51, 73 -> 63, 80 -> 66 (62 idle), 3 68 -> 71, 79 -> 93 (29 idle); 1 of f = 14336 66 -> 53, 74 -> 67 (53
// idle); 64 steps, 1 of f = 8192 37 -> 43 (43 idle).  And in several rounds that the
// fewest tiles leave idle for GG_FLEX_CUT_STEPS, with more than 64 rows per token tile: 128 steps, 5 experts of f = 14336, 24 rows
// 188 -> 200, 40 197 -> 200, 56 204 -> 203, 64 203 -> 204, 72 216 -> 209, 90 222 -> 211, 120 233 -> 218; 14 of them 588 -> 579; 11 of
// f = 6400 186 -> 198, 206 -> 210, 215 -> 217, 227 -> 223, 227 -> 220.
#define GG_FLEX_IDLE_STEPS 48
#define GG_FLEX_CUT_ROWS 64
GG_FN bool gg_up_cut(int N, int n_tok, int groups, int wgs, int KS, int split) {
    const int W = wgs * 8, total = n_tok * ((groups + 7) / 8), slots = (total + W - 1) / W * W;
    if (total == slots || !gg_sched(total, wgs, 0, KS, split).split) return false;
    if (slots == W) return (W - gg_flex_fill(n_tok, groups, wgs) * n_tok) * KS >= W * GG_FLEX_IDLE_STEPS;
    return (slots - total) * KS >= W * GG_FLEX_CUT_STEPS && N > GG_FLEX_CUT_ROWS * n_tok;
}
// Do the offsets allow tiles of 160 rows?  larger: an expert has more rows.
GG_FN bool gg_small_allowed(bool up, bool own_wide, int N, int E, bool larger) {
    return own_wide || (up && N <= GG_WIDE_MAX_ROWS * E) || !larger;
}
// Feature tiles per expert of the tiles of up to 160 rows, 0: the launch's own.  `active` experts with rows, in n_tok token tiles of 160
// rows or own_tok of the launch's, which have own_NT feature tiles per expert.
// only_wide (own tiles of 256 features): only for fewer rounds.  64 experts of f = 1408, own -> 160 rows, both one round 12 x 90
// rows 40 -> 44 us, 20 x 90 49 -> 51, 6 x 300 36 -> 54; both two, 200 tokens, Zipf 1.2, 98 -> 100..102, 44 x 40 92 -> 97; two and
// one 24 x 90 69 + 5 -> 61, 36 x 90 89 + 5 -> 81; three and two 64 x 28 128 + 5 -> 121.
// Where an expert has more of the launch's token tiles than of these, these are ahead whatever is idle (cut -> narrowed, 128 steps: 1
// x 160 rows of f = 14336 112 -> 92, 5 x 150 303 -> 264, 2 x 150 of f = 6400 106 -> 91) unless the last-level cache keeps the matrices of
// the experts in use and the launch's tiles are one round: two tiles of 5 blocks end before one of 10 does.  64 steps, own -> 160 rows: 2 x
// 150 rows of f = 8192 (134 MB) 47 -> 57, 4 x 150 (268 MB) 73 -> 66; 4, 8, 10 x 150 of f = 1792 (59, 117, 147 MB) 36, 44, 45 -> 51, 53,
// 54, 16 (235 MB) 69 -> 64; 128 steps, 1 x 150 of f = 6400 (105 MB) 42 -> 89.
// Reductions too short to cut, whatever the size of the matrices: 44 steps, 64 experts in the layer, own -> 160 rows: 12 x 150 rows
// 36 -> 43, 28 x 150 42 -> 53, 30 x 150 49 -> 54, 32 x 150 58 -> 56; 4 x 150 and 30 x 20 44 -> 54; 160 and 60 x 30 63 -> 75; in two
// rounds, 40 x 130 89 -> 70.
GG_FN int gg_small_tiles(bool up, int N, int E, int active, int n_tok, int own_tok, int own_NT, int FR, int wgs, int KS, int split,
                         bool only_wide) {
    if (KS < GG_SPLIT_KS && own_tok > n_tok && own_tok * own_NT <= wgs * 8) return 0;
    if (!up || N > GG_WIDE_MAX_ROWS * E) return gg_flex(N, n_tok, FR / 4, wgs, KS, split, only_wide);
    const int NT = gg_flex_fill(n_tok, FR / 4, wgs);
    const int W = wgs * 8;
    if (only_wide && (own_tok * own_NT + W - 1) / W <= (n_tok * NT + W - 1) / W) return 0;
    if (own_tok > n_tok)
        return own_tok * own_NT <= W && (long long)active * FR * KS <= GG_SMALL_MIN_FRAGS ? 0 : NT;
    return gg_up_cut(N, n_tok, FR / 4, wgs, KS, split) ? 0 : NT;
}
// HOST: is the projection run with the kernel that holds the tiles of 160 rows, too?  If they are to be expected with all experts in
// use; the other's tiles end without spills (77 tokens, second projection 151 us, 153 with the other body beside it).
// GG_UP_MAX_STEPS: both projections, own -> 160 rows in the first one with more steps: 192 steps, 8 experts of f = 8192 with 20 and 90
// rows 397 -> 394, 445 -> 438, 5 of them with 90 349 -> 301, skewed 501 -> 512; 256 steps, f = 14336 896 -> 875, 973 -> 935, skewed
// 1069 -> 1061.  Not taken for the skewed ones of 192 steps.
#define GG_UP_MAX_STEPS 128
GG_FN bool gg_small_expected(bool up, bool own_wide, int N, int E, int FR, int KS, int wgs) {
    if (N > GG_SMALL_ROWS * E || (long long)E * FR * KS < GG_SMALL_MIN_FRAGS) return false;
    const int split = gg_split_limit(up, KS, wgs);
    if (up && N <= GG_WIDE_MAX_ROWS * E)
        return KS <= GG_UP_MAX_STEPS && gg_flex((GG_FLEX_FEW_ROWS + 1) * E, E, FR / 4, wgs, KS, split, false) != 0;
    for (int n = E; n <= E + (own_wide ? N / GG_SMALL_ROWS : 0); n++)  // token tiles
        if (gg_flex(N, n, FR / 4, wgs, KS, split, !own_wide)) return true;
    return false;
}
// HOST: may such a first projection have pieces?  If not, its tiles are all left whole and no fix-up is launched (4.6 us where
// there is nothing to add).  least: experts in use, at least.  Cutting the launch's own tiles has to save GG_FIXUP_MIN_STEPS: 64 steps,
// tiles of 256 x 256, whole -> cut with fix-up: 1..4 experts of f = 1408 with 20..150 rows 25..35 -> 22..28 us; 47 steps saved at most, 6
// x 24 28 -> 26, 6 x 60 30 -> 30, 6 x 120 36 -> 34, 6 x 200 46 -> 39: not worth 4.6 us of every call with six experts per token (150
// of them); 8 x 100 35 -> 36, 8 x 225 47 -> 45, 10 x 180 45 -> 49.  Longer reductions always: 128 steps, 1 x 80 53 -> 26, 6 x 24 54 -> 39,
// 6 x 90 63 -> 49, 26 x 40 148 -> 125.
#define GG_FIXUP_MIN_STEPS 48
GG_FN bool gg_up_may_cut(int N, int E, int least, int own_rows, int own_NT, int FR, int KS, int wgs, bool only_wide) {
    const int W = wgs * 8, split = gg_split_limit(true, KS, wgs);
    const int own = (N + own_rows - 1) / own_rows, tok = (N + GG_SMALL_ROWS - 1) / GG_SMALL_ROWS;
    if (!split) return false;
    if ((only_wide || (long long)least * FR * KS <= GG_SMALL_MIN_FRAGS) &&
        (KS > GG_SPLIT_KS || (W - (own > least ? own : least) * own_NT) * KS >= W * GG_FIXUP_MIN_STEPS))
        return true;
    for (int n = tok > least ? tok : least; n <= E + N / GG_SMALL_ROWS; n++)
        if (gg_up_cut(N, n, FR / 4, wgs, KS, split)) return true;
    return false;
}
// Workgroup me of an XCD takes a different one of the round's 32 neighbours every round: the
// token tiles of an expert differ in length, and their period must not pick workgroups.
GG_FN int gg_round_slot(int n, int wgs, int xcd, int me) {
    return n * wgs * 8 + xcd * wgs + (int)((unsigned)(me + n) % (unsigned)wgs);
}

// Cut points of the left-over tiles' joint reduction (S = R tiles x KS steps) for the
// workgroups of one XCD: workgroup j covers [cut(j), cut(j+1)).  Pieces are multiples of
// `unit` steps (KS is one too) and no piece is shorter than the smallest multiple of `unit`
// that covers the `ns` LDS stages of the kernel's pipeline.
GG_FN int gg_piece_cut(int j, int S, int KS, int wgs, int unit, int ns) {
    const int minp = (ns + unit - 1) / unit * unit;
    int per = ((S + wgs - 1) / wgs + unit - 1) / unit * unit;
    per = per < 32 ? 32 : per;
    const int c = j * per;
    if (c >= S) return S;
    const int r = c % KS;
    if (r < minp) return c - r;
    if (KS - r < minp) return c + (KS - r);
    return c;
}

// Does every XCD start with a round of its own, an eighth of all rounds behind its neighbour's?  Tiles of
// an expert that has no other token tile wait for their weights from HBM, tiles of many rows are bound by the
// matrix cores' power: where both are there, they should be at work at the same time.  First projection, in
// step -> turned, at least 1 of 8 token tiles its expert's only one and at least 1 of 4 not: 16 experts, 4096 tokens Zipf
// 780 -> 734 us, 1531 tokens 429 -> 417, 8 experts, 1531 tokens 661 -> 625, 64 experts, 2000 tokens 210 -> 195; of 34 others,
// five shapes and three skews, 26 even to 10 % ahead, 8 behind by 1..3 %, most of them where no expert is much larger than another.
// Fewer only ones: 8 x 700 rows 1021 -> 1033, 4096 tokens 1473 -> 1471, its second projection 726 -> 733.  Fewer others:
// reductions of 128 and 256 steps, none 947..1014 -> 962..1044, 12 % 923 -> 1004, 17 % 1001 -> 1039, 21 % 1024 -> 1041, 22 %
// 967 -> 1005; of 64 steps none 465..510 -> 470..502, 9..12 % 507..531 -> 499..512, so there they do not count.  With fewer
// than 4 rounds: 2 rounds 342 -> 357.
#define GG_TURN_ROUNDS 4
#define GG_TURN_SHORT 64  // steps of the reduction
// ones: experts of one token tile, each NT of the total tiles.
GG_FN bool gg_turned(int ones, int total, int NT, int KS) {
    return ones * 8 * NT >= total && (KS <= GG_TURN_SHORT || (total - ones * NT) * 4 >= total);
}
// The XCD's first round.
GG_FN int gg_first_round(bool turned, int n_full, int xcd) {
    return turned && n_full >= GG_TURN_ROUNDS ? n_full * xcd / 8 : 0;
}
