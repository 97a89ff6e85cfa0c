"""The LDS row pitches of the local solves: the smallest pitch within 34 of the
number of lines that costs the fewest LDS cycles, recomputed from the access
pattern of k_fdm."""
import os
import re

import pytest

SRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                   "paper_2207_07098_amd", "csrc", "sem_gmres.hip")


def _cycles(values, served, banks):
    """LDS cycles of one instruction: `served` lanes at a time, each group as
    many cycles as the most distinct values that one bank holds."""
    total = 0
    for g in range(0, 64, served):
        used = {}
        for v in {v for v in values[g:g + served] if v is not None}:
            used[v % banks] = used.get(v % banks, 0) + 1
        total += max(used.values(), default=1)
    return total


def cost(ne, pitch, fp64, by_hi, banks):
    """Writes of a pass (results of every tile to the next direction's layout)
    and its reads; `banks` are of the value's size."""
    lines, steps = ne * ne, (ne + 3) // 4
    served = 16 if fp64 else 32
    total = 0
    for tile in range((lines + 15) // 16):
        for reg in range(steps if fp64 else 4):
            at = []
            for lane in range(64):
                col, q = 16 * tile + lane % 16, lane // 16
                row = q + 4 * reg if fp64 else 4 * q + reg
                lo, hi = col % ne, col // ne
                where = hi * pitch + lo + ne * row if by_hi else lo * pitch + ne * hi + row
                at.append(where if col < lines and row < ne else None)
            total += _cycles(at, served, banks)
        for s in range(steps):
            total += _cycles([min(4 * s + lane // 16, ne - 1) * pitch + 16 * tile + lane % 16
                              for lane in range(64)], served, banks)
    return total


def both(ne, pitch, fp64, by_hi):
    """With 32 banks of 4 bytes and with 64."""
    width = 2 if fp64 else 1
    return sum(cost(ne, pitch, fp64, by_hi, n // width) for n in (32, 64))


@pytest.mark.parametrize("name, fp64, by_hi", [("kHi64", True, True), ("kLo64", True, False),
                                               ("kHi32", False, True), ("kLo32", False, False)])
def test_tables_hold_the_cheapest_pitches(name, fp64, by_hi):
    with open(SRC) as f:
        table = [int(v) for v in re.search(name + r"\[12\] = \{([^}]*)\}", f.read()).group(1).split(",")]
    for ne, pitch in zip(range(5, 17), table):
        best = min(range(ne * ne, ne * ne + 34), key=lambda p: both(ne, p, fp64, by_hi))
        assert pitch == best, (ne, pitch, best)


def test_figures_of_the_comment():
    """NE = 10 in FP64: cycles of a pass with the table's pitches and with 112."""
    assert [both(10, p, True, h) // 2 for p, h in ((106, True), (105, False), (112, True), (112, False))] \
        == [168, 168, 198, 563]
