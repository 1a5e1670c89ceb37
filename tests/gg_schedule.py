"""The grouped GEMM's schedule (csrc/moe_gg_sched.h) on the host: the kernel's own functions behind
ctypes, and the work they deal out for a list of rows per expert."""
import ctypes as C
import os
import subprocess
import tempfile
from dataclasses import dataclass

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2402_07033_amd", "csrc")
SRC = r"""
#include "moe_gg_ring.h"
#include "moe_gg_sched.h"
extern "C" {
int split_limit(int up, int KS, int wgs) { return gg_split_limit(up != 0, KS, wgs); }
void sched(int total, int wgs, int xcd, int KS, int split, int* out) {
    const GgSched s = gg_sched(total, wgs, xcd, KS, split);
    out[0] = s.n_full; out[1] = s.left_lo; out[2] = s.R; out[3] = s.split;
}
int turned(int ones, int total, int NT, int KS) { return gg_turned(ones, total, NT, KS); }
int first_round(int turned, int n_full, int xcd) { return gg_first_round(turned != 0, n_full, xcd); }
int round_slot(int n, int wgs, int xcd, int me) { return gg_round_slot(n, wgs, xcd, me); }
int piece_cut(int j, int S, int KS, int wgs) { return gg_piece_cut(j, S, KS, wgs, GG_U, GG_NS); }
int up_cut(int N, int n_tok, int groups, int wgs, int KS, int split) { return gg_up_cut(N, n_tok, groups, wgs, KS, split); }
int up_may_cut(int N, int E, int least, int own_rows, int own_NT, int FR, int KS, int wgs, int only_wide) {
    return gg_up_may_cut(N, E, least, own_rows, own_NT, FR, KS, wgs, only_wide != 0);
}
}
"""
_lib = None


def lib():
    global _lib
    if _lib is None:
        with tempfile.TemporaryDirectory() as d:
            with open(os.path.join(d, "s.cpp"), "w") as fh:
                fh.write(SRC)
            so = os.path.join(d, "s.so")
            subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, "-o", so,
                            os.path.join(d, "s.cpp")], check=True)
            _lib = C.CDLL(so)
    return _lib


def schedule(total, wgs, xcd, KS, up):
    """gg_sched: rounds, the XCD's first left-over tile and their number, are they cut."""
    out = (C.c_int * 4)()
    lib().sched(total, wgs, xcd, KS, lib().split_limit(int(up), KS, wgs), out)
    return tuple(out)


@dataclass
class Branch:
    """Which way one projection of a call goes."""
    rounds: int      # of whole tiles
    left: int        # tiles of the last, incomplete round
    cut: bool        # ... in pieces
    turned: bool     # the XCDs start at different rounds
    once: set        # units of the tiles that are their expert's only one (weights past L2)
    shared: set      # units of the other tiles (weights kept in L2)


def tiles_of(rows, tile_rows):
    """Units (64 rows) of each token tile of an expert: dealt evenly, the first tiles take one more."""
    units = -(-rows // 64)
    tiles = -(-rows // tile_rows)
    return [units // tiles + (t < units % tiles) for t in range(tiles)]


def branch(counts, tile_rows, tile_features, weight_rows, KS, up, cus=256):
    """weight_rows: output features of the projection (2f, d); KS: steps of its reduction."""
    L, wgs = lib(), (cus + 7) // 8
    NT = weight_rows // tile_features
    per = [tiles_of(n, tile_rows) for n in counts if n]
    total = sum(map(len, per)) * NT
    n_full, _, _, cut = schedule(total, wgs, 0, KS, up)
    ones = sum(len(p) == 1 for p in per)
    left = total - n_full * wgs * 8
    turned = any(L.first_round(L.turned(ones, total, NT, KS), n_full, x) for x in range(8))
    return Branch(n_full, left, bool(cut) and left > 0, turned,
                  {u for p in per if len(p) == 1 for u in p}, {u for p in per if len(p) > 1 for u in p})


def dealt(total, KS, up, turned, wgs):
    """(tile, first step, steps) of every unit of work, workgroup by workgroup."""
    L, work = lib(), []
    for xcd in range(8):
        n_full, left_lo, R, split = schedule(total, wgs, xcd, KS, up)
        turn = L.first_round(int(turned), n_full, xcd)
        for me in range(wgs):
            mine = [(L.round_slot((n + turn) % n_full, wgs, xcd, me), 0, KS) for n in range(n_full)]
            if not split and (me + n_full) % wgs < R:
                mine.append((left_lo + (me + n_full) % wgs, 0, KS))
            if split and R:
                c0, c1 = L.piece_cut(me, R * KS, KS, wgs), L.piece_cut(me + 1, R * KS, KS, wgs)
                while c0 < c1:
                    n = min(c1, (c0 // KS + 1) * KS) - c0
                    mine.append((left_lo + c0 // KS, c0 % KS, n))
                    c0 += n
            work.append(mine)
    return work
