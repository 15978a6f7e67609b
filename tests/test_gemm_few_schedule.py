"""The hand-placed waits of the few-tile GEMM's loop, checked on its source: the
loads are issued in the order that the prologue and the step macro state, a wait
for n leaves the newest n in flight, and no fragment may be read from a stage
one of whose loads may still be among them.  (The compiler adds tighter waits
where it sees that a stage and a read may alias; the source has to hold without
them.)"""
import os
import re

import pytest

from conftest import ROOT

SRC = os.path.join(ROOT, "paper_2607_14557_amd", "csrc", "gemm_few.h")


def _source():
    s = open(SRC).read()
    step = re.search(r"#define FEW_STEP\(T, H, SC, SN, SF, BS\)(.*?)\n\n", s, re.S).group(1)
    tail = s[s.index(step) + len(step):]
    prologue = tail[:tail.index("FEW_READ(st0, 0, 0)")]
    tiles = re.findall(r"#define FEW_TILE\d\(T\) (.*)", tail)
    return step, prologue, tiles


def _wait(text, NJ):
    return eval(re.search(r"waitcnt_imm\(([^,]+), 15\)", text).group(1), {"NJ": NJ})


@pytest.mark.parametrize("NJ", [2, 4])
@pytest.mark.parametrize("n_tiles", [1, 2, 3, 8])
def test_no_read_of_a_stage_in_flight(NJ, n_tiles):
    step, prologue, tiles = _source()
    flying, held = [], {}            # loads in issue order; stage -> (K tile, half) last requested

    def issue_a(stage, tile, half, quarter):
        if quarter == 0:
            held[stage] = (tile, half)
        assert held[stage] == (tile, half)
        flying.extend([stage] * 2)

    def issue_b():
        flying.extend(["B"] * NJ)

    def wait(n):
        del flying[:max(0, len(flying) - n)]

    def read(stage, tile, half):
        assert held[stage] == (tile, half), "stage %s holds %s" % (stage, held[stage])
        assert stage not in flying, "%s read with %d of its loads in flight" % (stage, flying.count(stage))

    for lo, hi, what, args in re.findall(r"for \(int q = (\d); q < (\d); \+\+q\) FEW_([AB])\(([^)]*)\);", prologue):
        args = [a.strip() for a in args.split(",")]
        for q in range(int(lo), int(hi)):
            if what == "A":
                issue_a(args[0], int(args[1]), int(args[2]), q)
            else:
                issue_b()
    assert len(flying) == 24 + 4 * NJ
    wait(_wait(prologue, NJ))
    read("st0", 0, 0)
    # the step: its order of wait, read and loads
    order = [step.index(w) for w in ("if (ks == 3)", "FEW_READ(ks < 3 ? SC : SN", "FEW_A(SF, (T) + 1 + (H), (H) ^ 1, ks)",
                                     "if (ks < 2) FEW_B(")]
    assert order == sorted(order)
    for t in range(n_tiles):
        calls = re.findall(r"FEW_STEP\(T, (\d), (st\d), (st\d), (st\d), (\d)\)", tiles[t % 2])
        assert [c[0] for c in calls] == ["0", "1"]
        for h, sc, sn, sf, _ in calls:
            h = int(h)
            for ks in range(4):
                if ks == 3:
                    wait(_wait(step, NJ))
                read(sc if ks < 3 else sn, *((t, h) if ks < 3 else (t + h, h ^ 1)))
                issue_a(sf, t + 1 + h, h ^ 1, ks)
                if ks < 2:
                    issue_b()
