"""The counters that the waves of a one-workgroup solver share between barriers
(csrc/round_slots.h): every order in which the waves' steps can follow each
other is tried on a model of the loop, with the slots the kernels use and with
two slots by the round's parity, where a wave that is late to test the end of a
phase finds the next phase's rows."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
# per phase, per round but the last: how many rows each wave's losers are
PHASES = [[(1, 0), (0, 1)], [], [(1, 1)], []]
WAVES = 2


@pytest.fixture(scope="module")
def header(tmp_path_factory):
    d = tmp_path_factory.mktemp("slots")
    src, lib = d / "slots.cpp", d / "slots.so"
    src.write_text('#include "round_slots.h"\nextern "C" {\n'
                   "int slots() { return prot::kRoundSlots; }\n"
                   "int losers(int s) { return prot::losers_slot(s); }\n"
                   "int phase(int s) { return prot::phase_slot(s); }\n"
                   "int cleared(int s, int i) { return prot::cleared_by(s, i); }\n}\n")
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I",
                    os.path.join(ROOT, "paper_2203_03732_amd", "csrc"), str(src), "-o", str(lib)],
                   check=True)
    return ctypes.CDLL(str(lib))


def program(wave, rule):
    """A wave's steps: ('push', slot), ('clear', slot), ('rows', slot, expected),
    ('end', slot, whether the phase is over) and ('barrier',)."""
    n_slots, losers, phase, cleared = rule
    steps, s = [], 0
    for rounds in PHASES:
        steps += [("push", s), ("barrier",)]
        looking = WAVES
        for lost in rounds + [None]:
            steps.append(("rows", s, looking))
            if wave == 0:
                steps += [("clear", i) for i in range(n_slots) if cleared(s, i)]
            steps.append(("barrier",))
            if lost:
                steps += [("push", losers(s))] * lost[wave]
                looking = sum(lost)
            steps += [("barrier",), ("end", losers(s), lost is None)]
            s = losers(s) if lost else phase(s)
    return steps


def explore(rule):
    """Whether every interleaving reads what it should."""
    progs = [program(w, rule) for w in range(WAVES)]
    start = ((0,) * WAVES, (0,) * rule[0])
    seen, todo = {start}, [start]
    while todo:
        pcs, cnt = todo.pop()
        at = [p[i] if i < len(p) else None for p, i in zip(progs, pcs)]
        moves = []
        if all(a == ("barrier",) for a in at):
            moves.append((tuple(i + 1 for i in pcs), cnt))
        for w, a in enumerate(at):
            if a is None or a[0] == "barrier":
                continue
            c = list(cnt)
            if a[0] == "push":
                c[a[1]] += 1
            elif a[0] == "clear":
                c[a[1]] = 0
            elif a[0] == "rows" and c[a[1]] != a[2]:
                return False
            elif a[0] == "end" and (c[a[1]] == 0) != a[2]:
                return False
            moves.append((tuple(i + (v == w) for v, i in enumerate(pcs)), tuple(c)))
        for m in moves:
            if m not in seen:
                seen.add(m)
                todo.append(m)
    return True


def test_every_order(header):
    assert explore((header.slots(), header.losers, header.phase, header.cleared))


def test_parity_is_not_enough():
    assert not explore((2, lambda s: s ^ 1, lambda s: s ^ 1, lambda s, i: i != s))


def test_clearing_less_is_not_enough():
    three = lambda s: (s + 1) % 3  # noqa: E731
    assert not explore((3, three, lambda s: (s + 2) % 3, lambda s, i: i == (s + 2) % 3))
