"""The batch worker's words in LDS.  Its loop is read from the source as a
sequence of block barriers, writes by thread 0 and reads by every wave, along
every path through its branches: a word is never written and read between the
same two barriers, so no wave can see the value meant for another step."""
import itertools
import os
import re

HERE = os.path.dirname(os.path.abspath(__file__))
SOURCE = os.path.join(os.path.dirname(HERE), "paper_2401_04701_amd", "csrc", "hr_batch.hip")

TOKEN = re.compile(r"""(?P<barrier>__syncthreads\(\))
    | uni(?:64)?\((?P<read>s_\w+)\)
    | (?P<write>\bs_\w+)\s*=(?!=)
    | (?P<branch>\bif\s*\((?!threadIdx\.x\s*==\s*0\)))
    | (?P<open>\{) | (?P<close>\})""", re.X)


def body(text, head):
    """The brace block that follows `head`."""
    at = text.index("{", text.index(head))
    depth = 0
    for i in range(at, len(text)):
        depth += {"{": 1, "}": -1}.get(text[i], 0)
        if depth == 0:
            return text[at + 1:i]
    raise ValueError(head)


def events(text):
    """[(kind, name, branches it is under)] in source order."""
    out, under, ids, pending = [], [], itertools.count(), None
    for m in TOKEN.finditer(text):
        kind = m.lastgroup
        if kind == "branch":
            pending = next(ids)          # its own block, if it opens one
            continue
        if kind == "open":
            under.append(pending)
            pending = None
        elif kind == "close":
            under.pop()
        else:
            out.append((kind, m.group(kind), tuple(b for b in under if b is not None)))
    return out


def loop_events():
    with open(SOURCE) as f:
        text = re.sub(r"//[^\n]*", "", f.read())
    whole = body(text, "void batch_loop(")
    loop = body(whole, "for (;;)")
    return events(whole[:whole.index("for (;;)")]), events(loop)


def paths(ev):
    """Every choice of branches taken."""
    branches = sorted({b for e in ev for b in e[2]})
    for taken in itertools.product([False, True], repeat=len(branches)):
        on = {b for b, t in zip(branches, taken) if t}
        yield [(k, n) for k, n, under in ev if set(under) <= on]


def conflict(seq):
    """A word written and read with no barrier in between, or None."""
    seen = {"read": set(), "write": set()}
    for kind, name in seq:
        if kind == "barrier":
            seen = {"read": set(), "write": set()}
            continue
        other = "write" if kind == "read" else "read"
        if name in seen[other]:
            return name
        seen[kind].add(name)
    return None


def test_the_reader_finds_a_missing_barrier():
    b, w, r = ("barrier", ""), ("write", "s_x"), ("read", "s_x")
    assert conflict([w, b, r, b, w, b, r]) is None
    assert conflict([w, b, r, w]) == "s_x" and conflict([w, r]) == "s_x"
    ev = events("if (threadIdx.x == 0) { s_a = 1; } __syncthreads(); if (q && uni(s_a)) { "
                "__syncthreads(); }")
    assert [e[0] for e in ev] == ["write", "barrier", "read", "barrier"]
    assert sorted(len(p) for p in paths(ev)) == [3, 4]


def test_no_word_is_written_and_read_between_two_barriers():
    first, loop = loop_events()
    words = {n for k, n, _ in loop if k == "read"}
    assert len(words) >= 2 and words == {n for k, n, _ in loop if k == "write"}
    for start in paths(first):
        for one in paths(loop):
            for two in paths(loop):
                assert conflict(start + one + two) is None, conflict(start + one + two)
