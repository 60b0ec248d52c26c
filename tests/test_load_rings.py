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


def _mid_instances():
    """(waves, blocks, gate/up) of every gemm_bf16_mid_k that the library launches."""
    out = {(int(a), int(b), g == "true") for a, b, g in re.findall(r"launch_mid<(\d), (\d), (true|false)", SRC)}
    for name, glu in (("launch_mid_glu", True), ("launch_mid_rest", False)):
        body = SRC[SRC.index(f"static hipError_t {name}("):]
        body = body[:body.index("\n}\n")]
        out |= {(int(a), int(b), glu) for a, b in re.findall(r"TLT_MID\((\d), (\d)\)", body)}
    return sorted(out)


def _mid_ring(nw, wtn, glu):
    """(slots, loads per wave and step, of them under slice 3), as launch_mid and the kernel have them."""
    idle = 4 * wtn % nw != 0
    fit = ((159 if glu else 160 - idle) * 1024) // ((32 * nw + 32 * wtn) * 128)
    L = 4 + -(-4 * wtn // nw)
    return min(fit, 6), L, (L + 3) // 4


def test_the_wave_per_32_rows_instances_are_found():
    found = _mid_instances()
    assert len(found) >= 35 and {nw for nw, *_ in found} == set(range(2, 9)) and {wtn for _, wtn, _ in found} == set(range(2, 8))
    for text in ("S = kFit < 6 ? kFit : 6", "kFit = (GLU ? 159 * 1024 : 160 * 1024 - (kIdle ? 1024 : 0)) / kSlot", "LA = 4, LB = (BN / 8 + NW - 1) / NW, L = LA + LB",
                 "constexpr int Q3 = (L + 3) / 4;"):
        assert text in SRC, text


@pytest.mark.parametrize("nw,wtn,glu", _mid_instances())
def test_a_k_step_has_landed_before_it_is_read_by_a_wave_per_32_rows(nw, wtn, glu):
    """The kernel's issue order (steps 0 .. S - 2 whole and the first Q3 loads of the next in the prologue; in step t the rest of step t + S - 1 under slices 0
    to 2, then the wait, then the first Q3 of step t + S) and its two waits; and a slot is refilled only behind the barrier after its last read."""
    S, L, Q3 = _mid_ring(nw, wtn, glu)
    first, loop = re.search(r"waitcnt\(vmcnt_imm\((.*?)\)\);   // step 0 has landed", SRC), re.search(r"waitcnt\(vmcnt_imm\((.*?)\)\);   // step t \+ 1 has landed", SRC)
    value = lambda m: eval(m.group(1), {"S": S, "L": L, "Q3": Q3})
    assert S >= 3 and value(first) < 64
    order = [t for t in range(S - 1) for _ in range(L)] + [S - 1] * Q3
    last = lambda step: max(i for i, t in enumerate(order) if t == step)
    assert value(first) <= len(order) - 1 - last(0)
    for t in range(4 * S):
        # slices 0 .. 2 of step t: slot t % S is read, the slot of step t - 1 is refilled (its reads ended before the barrier of step t - 1)
        share = sum((kk + 1) * (L - Q3) // 3 - kk * (L - Q3) // 3 for kk in range(3))
        assert share == L - Q3 and (t + S - 1) % S == (t - 1) % S
        order += [t + S - 1] * share
        assert value(loop) <= len(order) - 1 - last(t + 1), t
        order += [t + S] * Q3           # slice 3, behind the barrier: slot t % S, whose last fragments are in registers
