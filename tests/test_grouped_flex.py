"""Feature tiles of the grouped GEMM's tiles of up to 160 rows (gg_flex in csrc/moe_gg_sched.h), replayed on the CPU with the kernel's own functions."""
import ctypes as C
import os
import subprocess
import tempfile

import pytest

import gg_schedule
import paper_2402_07033_amd as moe

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = r"""
#include "moe_gg_ring.h"
#include "moe_gg_sched.h"
extern "C" {
int limit(int up, int KS, int wgs) { return gg_split_limit(up != 0, KS, wgs); }
int flex(int N, int n_tok, int groups, int wgs, int KS, int split, int only_wide) {
    return gg_flex(N, n_tok, groups, wgs, KS, split, only_wide != 0);
}
int fill(int n_tok, int groups, int wgs) { return gg_flex_fill(n_tok, groups, wgs); }
int is_cut(int total, int wgs, int KS, int split) { return gg_sched(total, wgs, 0, KS, split).split; }
}
"""


@pytest.fixture(scope="module")
def L():
    with tempfile.TemporaryDirectory() as d:
        with open(os.path.join(d, "s.cpp"), "w") as fh:
            fh.write(SRC)
        so = os.path.join(d, "s.so")
        subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I",
                        os.path.join(ROOT, "paper_2402_07033_amd", "csrc"), "-o", so, os.path.join(d, "s.cpp")],
                       check=True)
        yield C.CDLL(so)


def feature_tiles(L, N, n_tok, groups, wgs, KS, up, only_wide):
    return L.flex(N, n_tok, groups, wgs, KS, L.limit(int(up), KS, wgs), int(only_wide))


@pytest.mark.parametrize("groups", [2048, 448, 200, 64, 44, 16, 4, 1])
@pytest.mark.parametrize("wgs", [32, 5, 1])
def test_tiles_fill_their_rounds(L, groups, wgs):
    W = 8 * wgs
    for n_tok in range(0, 170):
        NT, least = L.fill(n_tok, groups, wgs), -(-groups // 8)
        assert least <= NT <= max(groups // 3, least)
        widths = {(nt + 1) * groups // NT - nt * groups // NT for nt in range(NT)}
        assert min(widths) >= 1 and max(widths) <= 8
        slots = -(-(n_tok * least) // W) * W
        assert n_tok * NT <= slots
        if n_tok:  # one tile more per token tile would not fit, or be of fewer than three groups
            assert n_tok * (NT + 1) > slots or 3 * (NT + 1) > groups


# groups of 4 fragment rows per expert: 448 / 64 (d 4096, f 14336), 200, 44 / 32 (d 2048, f 1408), 8, 4
@pytest.mark.parametrize("groups", [448, 200, 64, 44, 32, 8, 4])
@pytest.mark.parametrize("KS", [8, 44, 64, 128, 200, 448])
@pytest.mark.parametrize("wgs", [32, 5])
def test_tiles_hold_every_group_once(L, groups, KS, wgs):
    W = 8 * wgs
    for n_tok in list(range(0, 17)) + [31, 58, 63, 64]:
        for up in (0, 1):
            least = -(-groups // 8)
            total, rounds = n_tok * least, -(-(n_tok * least) // W)
            for only_wide, rows in ((False, 20), (False, 90), (True, 20), (True, 90)):
                NT = feature_tiles(L, rows * n_tok, n_tok, groups, wgs, KS, up, only_wide)
                if NT == 0:  # the launch's own tiles: nothing to do, as wide, full enough, or cut
                    assert (n_tok == 0 or only_wide or (rows <= 32 and (rounds * W - total) * 10 <= 3 * W)
                            or L.is_cut(total, wgs, KS, L.limit(up, KS, wgs)))
                    continue
                assert least <= NT <= groups and NT == L.fill(n_tok, groups, wgs)
                edges = [nt * groups // NT for nt in range(NT + 1)]
                widths = [b - a for a, b in zip(edges, edges[1:])]
                assert sum(widths) == groups and min(widths) >= 1 and max(widths) <= 8
                assert n_tok * NT <= rounds * W  # narrower tiles, no more rounds
                assert not only_wide or groups > 4 * NT
                if NT > least:
                    assert groups >= 3 * NT


@pytest.mark.parametrize("n_tok,groups,KS,up,only_wide,want", [
    # 8 experts, d 4096, f 14336: 448 tiles of 8 groups are 1.75 rounds, 512 of 7 are two; the second
    # projection's 64 are better cut
    (8, 448, 128, 1, False, 64), (8, 448, 128, 1, True, 64), (8, 64, 448, 0, False, 0), (8, 64, 448, 0, True, 0),
    # 16 experts, f 6400: 1.56 rounds -> two; half a round of 8 groups -> one of 4, which the 256-feature tiles are
    (16, 200, 128, 1, False, 32), (16, 64, 200, 0, False, 16), (16, 64, 200, 0, True, 0),
    # 64 experts, f 1408: 1.5 rounds of 6 tiles -> two of 8; a full round
    (64, 44, 64, 1, True, 8), (64, 32, 44, 0, False, 4),
    # a tenth of a second round is cut; one expert cannot fill a round with tiles of 3 groups
    (5, 448, 128, 1, False, 0), (1, 448, 128, 1, False, 0), (0, 448, 128, 1, False, 0)])
def test_rule(L, n_tok, groups, KS, up, only_wide, want):
    assert feature_tiles(L, 90 * n_tok, n_tok, groups, 32, KS, up, only_wide) == want
    # with few rows the 512-feature tiles stay if they fill 0.7 of the last round, the others do not
    few = feature_tiles(L, 32 * n_tok, n_tok, groups, 32, KS, up, only_wide)
    full = n_tok * -(-groups // 8) % 256 * 10 >= 7 * 256 or n_tok * -(-groups // 8) % 256 == 0
    assert few == (0 if full and not only_wide else want)


# d, f, rows of the experts in use, experts -> feature tiles of 160 rows per expert, 0: the launch's own; each line is a
# measurement that stands beside the rule
MIXTRAL, SIXTEEN, SIXTYFOUR = (4096, 14336, 8), (4096, 6400, 16), (2048, 1408, 64)
FEW = [
    (MIXTRAL, [90], 0), (MIXTRAL, [160], 149), (MIXTRAL, [300], 128), (MIXTRAL, [24] * 2, 128),
    (MIXTRAL, [24] * 5, 102), (MIXTRAL, [64] * 5, 102), (MIXTRAL, [72] * 5, 0), (MIXTRAL, [150] * 5, 102),
    (MIXTRAL, [90] * 8, 64), (MIXTRAL, [20] * 8, 64),
    (SIXTEEN, [90], 0), (SIXTEEN, [150], 0), (SIXTEEN, [300], 0), (SIXTEEN, [24] * 2, 0), (SIXTEEN, [90] * 2, 0),
    (SIXTEEN, [150] * 2, 66), (SIXTEEN, [90] * 3, 66), (SIXTEEN, [24] * 11, 46), (SIXTEEN, [90] * 11, 0),
    (SIXTYFOUR, [90], 0), (SIXTYFOUR, [24] * 6, 0), (SIXTYFOUR, [300] * 6, 0), (SIXTYFOUR, [150] * 12, 0),
    (SIXTYFOUR, [150] * 20, 0), (SIXTYFOUR, [90] * 24, 10), (SIXTYFOUR, [28] * 64, 8),
    ((2048, 8192, 16), [150] * 2, 0), ((2048, 8192, 16), [150] * 4, 64),
    ((2048, 1792, 32), [150] * 8, 0), ((2048, 1792, 32), [150] * 16, 16),
    ((4096, 1408, 64), [90] * 24, 10), ((4096, 1408, 64), [90] * 47, 0), ((4096, 1408, 64), [40] * 44, 0)]


def first(counts, d, f, k=1):
    return moe.moe_expert_ffn_tiles(counts, d, f, path=moe.MOE_FFN_GROUPED, k=k)["up"]


def small(t):
    return t["feature_tiles"] if t["rows"] == 160 else 0


@pytest.mark.parametrize("shape,rows,want", FEW)
def test_first_projection_of_few_experts(shape, rows, want):
    d, f, E = shape
    counts = rows + [0] * (E - len(rows))
    got = first(counts, d, f)
    assert small(got) == want
    assert got["fixup"] or not got["pieces"]
    # what the launch's own tiles are cut into needs the fix-up, whatever is known of the experts in use
    told = first(counts, d, f, k=min(len(rows), 8))
    assert small(told) == want and (told["pieces"] == got["pieces"] or (f % 256 and d // 32 == 64))


def test_first_projection_in_as_many_rounds_of_its_own_tiles():
    # 200 tokens on 64 experts, Zipf 1.2: 46 tiles of 256 rows x 11 fill two rounds, as 48 of 160 x 10 would
    rows = [194, 169, 147, 108, 95, 81, 50, 49, 45, 32, 34, 21, 21, 16, 14, 9, 14, 10, 13, 6, 5, 6, 6, 6, 2, 5, 6, 6, 4, 4,
            2, 5, 1, 2, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1]
    d, f, E = SIXTYFOUR
    assert small(first(rows + [0] * (E - len(rows)), d, f)) == 0
    assert small(first(rows + [1] * 6 + [0] * 12, d, f)) == 9  # three rounds


@pytest.mark.parametrize("d,f,E", [MIXTRAL, SIXTEEN, SIXTYFOUR, (2048, 1792, 32), (4096, 1408, 64)])
@pytest.mark.parametrize("least", [1, 2, 6])
def test_no_fixup_where_pieces_are_ruled_out(d, f, E, least):
    """Where no fix-up is launched, no number of token tiles is one that the rule would rather cut."""
    L, KS, FR, wgs = gg_schedule.lib(), d // 32, f // 8, 32
    wide = f % 256 == 0
    rows, NT, split = (128, FR // 32, L.split_limit(1, KS, wgs)) if wide else (256, FR // 16, L.split_limit(1, KS, wgs))
    launched = set()
    for N in list(range(73, 400, 9)) + list(range(400, 96 * E, 97)):
        may = bool(L.up_may_cut(N, E, least, rows, NT, FR, KS, wgs, int(not wide)))
        launched.add(may)
        if may:
            continue
        for n in range(max(least, -(-N // 160)), E + N // 160 + 1):
            assert not L.up_cut(N, n, FR // 4, wgs, KS, split), (N, n)
        assert wide or (KS == 64 and (256 - max(least, -(-N // 256)) * NT) * KS < 256 * 48)
        assert not wide or least * FR * KS > 128 << 10 or (256 - max(least, -(-N // 128)) * NT) * KS < 256 * 48
    assert (True in launched) == (wide or KS > 64 or least < 6)


@pytest.mark.parametrize("rows,want", [
    # 64 experts of f = 1408, second projection (44 steps): one round of the launch's own tiles, of which 150 rows are
    # two that end before one of 160 rows does; two rounds; no expert with more of them
    ([150] * 12, 0), ([150] * 28, 0), ([160] + [30] * 60, 0), ([150] * 4 + [20] * 30, 0), ([130] * 40, 6),
    ([128] * 12, 10), ([90] * 24, 10)])
def test_second_projection_too_short_to_cut(rows, want):
    d, f, E = SIXTYFOUR
    got = moe.moe_expert_ffn_tiles(rows + [0] * (E - len(rows)), d, f, path=moe.MOE_FFN_GROUPED)["down"]
    assert small(got) == want and not got["fixup"]
