"""The grouped GEMM's LDS ring, replayed on the CPU with the kernel's own constants
(csrc/moe_gg_ring.h): its waves meet only at the barriers, so whatever has to happen in one wave
before something in another needs a barrier between the two.  Two such pairs per ring slot: every
wave's reads of a stage have returned before any wave requests the next contents of the slot, and
every wave's share of a stage has arrived before any wave reads it."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2402_07033_amd", "csrc")
PRINT = r"""
#include <cstdio>
#include "moe_gg_ring.h"
int main() { std::printf("%d %d %d %d %d %d\n", GG_NS, GG_U, GG_LA, GG_WIDE_LA, GG_AHEAD, GG_BARRIER_STEPS); }
"""


@pytest.fixture(scope="module")
def ring(tmp_path_factory):
    d = tmp_path_factory.mktemp("ring")
    (d / "p.cpp").write_text(PRINT)
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, "-o", str(d / "p"), str(d / "p.cpp")], check=True)
    out = subprocess.run([str(d / "p")], check=True, capture_output=True, text=True).stdout
    return dict(zip(("ns", "u", "la", "wide_la", "ahead", "barrier"), map(int, out.split())))


def _unordered(ns, ahead, la, barrier, steps=64):
    """Stages that no barrier orders: ("refill", s) requested while another wave may still read
    the slot's previous contents, ("read", s) read before its arrival.  A wave's program: step k waits for the requests
    of step k - la, meets the barrier if k % barrier == 0, requests stage k + ahead, and reads
    stage k + 1, whose last read returns at the end of step k + 1."""
    pos, bars = 1, [1]                         # barrier of the prologue
    requested, end = {}, {}
    arrived = {s: 0 for s in range(ahead)}     # the prologue's own requests and wait
    reads = {0: 2}                             # program positions, the same in every wave
    pos = 2
    for k in range(steps):
        pos += 1
        if k >= la:
            arrived[k - la + ahead] = pos
        if k % barrier == 0:
            pos += 1
            bars.append(pos)
        pos += 1
        requested[k + ahead] = reads[k + 1] = pos
        pos += 1
        end[k] = pos                           # the reads of stage k have returned

    def ordered(first, second):
        return any(first < b < second for b in bars)

    bad = [("refill", s) for s, p in requested.items() if s >= ns and not ordered(end[s - ns], p)]
    bad += [("read", s) for s, p in reads.items() if s in arrived and not ordered(arrived[s], p)]
    return bad


@pytest.mark.parametrize("which", ["la", "wide_la"])
def test_ring_order(ring, which):
    assert ring["u"] % ring["barrier"] == 0   # a tile starts at a barrier step
    assert _unordered(ring["ns"], ring["ahead"], ring[which], ring["barrier"]) == []


def test_replay_finds_what_it_looks_for(ring):
    """One stage more ahead: an odd step refills what another wave may still be reading.  One
    step deeper weight ring than the stages allow: a stage is read before it is published."""
    ns, bar = ring["ns"], ring["barrier"]
    late = _unordered(ns, ns - 1, 3, bar)
    assert late and all(w == "refill" and (s - (ns - 1)) % 2 == 1 for w, s in late)
    assert any(w == "read" for w, _ in _unordered(ns, ns - 2, ns - 3, bar))
