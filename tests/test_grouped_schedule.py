"""The grouped GEMM's schedule, replayed on the CPU with the kernel's own functions
(csrc/moe_gg_sched.h): every step of every tile is dealt exactly once."""
import pytest

import gg_schedule as gs
from test_gpu_grouped_units import ROUNDS, long_branch


@pytest.mark.parametrize("wgs", [32, 5])
@pytest.mark.parametrize("KS", [8, 64, 128, 448])
@pytest.mark.parametrize("up", [True, False])
def test_every_step_is_dealt_once(wgs, KS, up):
    W = 8 * wgs
    for rounds in (0, 1, 3, 4, 7, 8, 11):
        for left in sorted({0, 1, 7, W // 16, W // 4, W // 2 + 3, 5 * W // 8, 11 * W // 16, W - 1}):
            total = rounds * W + left
            for turned in (False, True):
                work = gs.dealt(total, KS, up, turned, wgs)
                steps = {}
                for mine in work:
                    pieces = [m for m in mine if m[2] < KS]
                    # the kernel has two scratch slots per workgroup; a piece covers its ring's 8 stages
                    assert len(pieces) <= 2 and all(n >= 8 and n % 4 == 0 for _, _, n in pieces)
                    for tile, lo, n in mine:
                        steps.setdefault(tile, []).append((lo, n))
                assert sorted(steps) == list(range(total))
                for parts in steps.values():
                    at = 0
                    for lo, n in sorted(parts):
                        assert lo == at
                        at += n
                    assert at == KS


@pytest.mark.parametrize("up", [True, False])
@pytest.mark.parametrize("KS", [64, 128, 448])
def test_a_small_left_over_is_cut_behind_any_number_of_rounds(up, KS):
    """A tenth of a round left whole costs nearly a tile's time, however many rounds came before."""
    for rounds in (0, 1, 7, 8, 9, 25, 56):
        assert gs.schedule(rounds * 256 + 24, 32, 0, KS, up)[3]
    for rounds in (0, 8):    # and nearly a whole round stays whole
        assert not gs.schedule(rounds * 256 + 200, 32, 0, KS, up)[3]


@pytest.mark.parametrize("counts,KS,turned", [
    ([200] * 16, 128, False), ([200] * 16, 64, True),               # every expert has one tile
    ([600] + [200] * 15, 128, False), ([600] + [200] * 15, 64, True),  # 3 of 18 tiles are a larger expert's
    ([1500] + [130] * 15, 128, True),                               # 6 of 21
    ([1800] * 14 + [100], 128, False), ([1800] * 14 + [100], 64, False)])   # 1 of 113 is an only one
def test_turned_rounds_need_tiles_of_either_kind(counts, KS, turned):
    got = gs.branch(counts, 256, 256, 32768, KS, True)
    assert got.rounds >= 4 and got.turned == turned
    # and never with fewer than four rounds
    assert not gs.branch(counts[:2], 256, 256, 8192, KS, True).turned


@pytest.mark.parametrize("tile_rows", [256, 192, 128])
@pytest.mark.parametrize("up", [True, False])
def test_gpu_cases_reach_every_branch(up, tile_rows):
    """The cases that the GPU runs in rounds, per tile shape and projection: every number of units with either
    load policy, cut and whole left-over tiles, turned rounds, few and many rounds."""
    cases = [long_branch(n, up) for n, c in ROUNDS.items() if c[2] == tile_rows]
    for n, c in ROUNDS.items():
        b = long_branch(n, up)
        assert (b.rounds, b.cut, b.turned) == c[4], n
    units = set(range(1, tile_rows // 64 + 1))
    assert set().union(*(b.once for b in cases)) == units
    # (dealt evenly, a tile of one unit among several is there in the two-unit tiles only)
    assert set().union(*(b.shared for b in cases)) == units - ({1} if tile_rows > 128 else set())
    assert {b.cut for b in cases} == {b.turned for b in cases} == {True, False}
    assert min(b.rounds for b in cases) < 4 and max(b.rounds for b in cases) >= 8
