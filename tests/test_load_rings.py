"""The tiled GEMM's slot rings: loads retire in order, and before a K tile is read the kernel waits until at most kInFlight are outstanding.  Here
the order in which a wave issues its loads is written out for every instance that the library launches, and the wait checked
against it at every K step, the first ones included."""
import os
import re

import pytest

import paper_2511_16665_amd

SRC = open(os.path.join(os.path.dirname(paper_2511_16665_amd.__file__), "csrc", "gemm.hip")).read()


def _instances():
    """(SA, SB, LA, LB) of every launch_pipe<...> and launch_rowmax<...> in the source."""
    out = set()
    for name, args in re.findall(r"(launch_pipe|launch_rowmax)<([\d, ]+)", SRC):
        a = [int(x) for x in args.strip(", ").split(",")]
        wgm, wgn, wtm, wtn, sa, sb = a[:6] if name == "launch_pipe" else (*a[:3], 4, *a[3:5])
        waves = wgm * wgn
        out.add((sa, sb, 32 * wtm * wgm // 8 // waves, 32 * wtn * wgn // 8 // waves))
    return sorted(out)


def _issue_order(SA, SB, LA, LB, steps):
    """Loads in issue order as (operand, K tile); marks[t] = how many are issued when step t waits for tile t + 1."""
    order = [("A", 0)] * LA + [("B", 0)] * LB                                       # prologue
    for t in range(1, SA - 1):
        order += [("A", t)] * LA
    for t in range(1, SB - 1):
        order += [("B", t)] * LB
    order += [("B", SB - 1)] * (LB // 2)
    marks = []
    for t in range(steps):
        order += [("B", t - 1 + SB)] * (LB - LB // 2) + [("A", t - 1 + SA)] * LA
        marks.append(len(order))
        order += [("B", t + SB)] * (LB // 2)
    return order, marks


def test_the_instances_are_found():
    assert len(_instances()) >= 8 and any(sa == 4 for sa, *_ in _instances())


@pytest.mark.parametrize("SA,SB,LA,LB", _instances())
def test_a_k_tile_has_landed_before_it_is_read(SA, SB, LA, LB):
    a, b = re.search(r"constexpr int kInFlightA = (.*?), kInFlightB = (.*?);", SRC).groups()
    allowed = min(eval(e, {"SA": SA, "SB": SB, "LA": LA, "LB": LB}) for e in (a, b))
    order, marks = _issue_order(SA, SB, LA, LB, 3 * (SA + SB))
    for t, issued in enumerate(marks):
        behind = min(issued - 1 - max(i for i, load in enumerate(order) if load == (op, t + 1)) for op in "AB")
        assert allowed <= behind, (t, allowed, behind)
