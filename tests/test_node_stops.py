"""Where the waves of a node-weight fit leave after a stop (nodes.hip: Book::run,
Members::run), emulated on the CPU: the bookkeeping wave, a generation behind, and
the members' waves have to leave at the same generation, wherever a launch begins
and ends, whatever the node set, and whenever the stop is found -- a wave that
left by itself would pair the others' barriers with its own.

The waves run in lockstep from barrier to barrier; what the books write during a
generation is seen by a member either before or after, so both are tried.
"""
import itertools
import os
import re

import pytest

from paper_1906_10598_amd import build

LOOK = int(re.search(r"kAbandonLook = (\d+);", open(os.path.join(build.CSRC, "nodes.hip")).read()).group(1))
NEVER = 1 << 30
STOP, ABANDONED = 4, 1 << 16


def leaves(g0, g1, first2, stops, stop_at, flag, early):
    """Generations at which the books and the members leave, and the flags found.

    first2: generation (a multiple of 16) from which the smallest set is in use;
    early: a member reads what the books write in the same generation.
    """
    stop, abandoned = [0, 0], NEVER
    f1 = f2 = 0
    left = {}
    kind = 2 if g0 >= first2 else 1

    def step(g):
        nonlocal abandoned
        flags = flag if g >= stop_at else 0
        writes = [(g & 1, flags)]
        return flags, writes, (g if flags == ABANDONED else NEVER)

    for g in range(g0, g1):
        if g == first2:
            kind = 2
        # the books
        writes, new_abandoned, book_leaves = [], NEVER, False
        if f2:
            book_leaves = stops or kind < 2 or not g & (LOOK - 1)
        elif g > g0:
            f1, writes, new_abandoned = step(g - 1)
        # the members: on what is written before this generation, or also during it
        seen, seen_ab = list(stop), abandoned
        if early:
            for k, v in writes:
                seen[k] = v
            seen_ab = min(seen_ab, new_abandoned)
        if kind == 2 and not stops:
            member_leaves = not g & (LOOK - 1) and seen_ab <= g - 2
        else:
            member_leaves = g > g0 + 1 and seen[g & 1] != 0
        for k, v in writes:
            stop[k] = v
        abandoned = min(abandoned, new_abandoned)
        if book_leaves:
            left["books"] = g
        if member_leaves:
            left["members"] = g
        if left:
            break
        f2 = f1
    else:
        if not f2:
            flags, writes, ab = step(g1 - 1)
            stop[writes[0][0]] = flags
            abandoned = min(abandoned, ab)
        left = {"books": g1, "members": g1}
    g = left.get("members", left.get("books"))
    flags = stop[g & 1]
    if g == g1 and not (g1 - g0 > 1 and flags):
        flags = stop[(g1 - 1) & 1]
    if abandoned != NEVER:
        flags = ABANDONED
    return left, flags


@pytest.mark.parametrize("stops", [False, True])
@pytest.mark.parametrize("early", [False, True])
def test_all_waves_leave_together(stops, early):
    for g0, ngen, first2 in itertools.product((*range(0, 34), LOOK - 1, LOOK, LOOK + 1), (1, 2, 3, 7, 8, 9, 16, 17, 40, LOOK + 1, 2 * LOOK),
                                            (0, 16, 32, 48, NEVER)):
        g1 = g0 + ngen
        for stop_at in list(range(g0, g1)) + [NEVER]:
            # without a stop rule nothing but the abandonment stops a fit
            for flag in (STOP, ABANDONED) if stops else (ABANDONED,):
                left, flags = leaves(g0, g1, first2, stops, stop_at, flag, early)
                assert set(left) == {"books", "members"}, (g0, g1, first2, stop_at, flag)
                assert left["books"] == left["members"]
                assert flags == (flag if stop_at < g1 else 0), (g0, g1, first2, stop_at, flag)
                if stop_at < g1:
                    assert left["books"] <= max(stop_at + 2 + LOOK, g1 if stop_at + 2 >= g1 else 0)
