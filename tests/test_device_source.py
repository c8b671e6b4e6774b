"""A rule of the device code that no compiler checks: where the words of a task's descriptor are looked up."""
import os
import re

import pytest

from paper_2604_15379_amd import build as B

KERNELS = os.path.join(os.path.dirname(B.__file__), "csrc", "kernels.hip.inc")
# look-ups, and the functions that make them
LOOKUP = re.compile(r"\b(?:task|op)\s*\[|\btask\.u64\(|\bop\.hot\(|\b(?:takes_input|store_buf|wait_event|wait_gemm|trace_begin|signal_event|finish_task)\(")
UNIFORM = re.compile(r"\b(?:sreg|uni|uni64|uni_ptr|__builtin_amdgcn_readfirstlane|__builtin_amdgcn_ballot_w64)\(")   # one value for all lanes, whatever is in it
NAME = re.compile(r"\s*[*&]?(\w+)\s*=(?!=)(.*)", re.S)
DECLARATION = re.compile(r"[;{}(]\s*(?:const\s+)?(?:int|bool|auto|float|size_t|u16|uint32_t)\b\s*\*?\s*(?:const\s+)?(?=\w+\s*=[^=])")
CONDITION = re.compile(r"\b(?:if|for|while)\s*(?=\()")
PAIR = {"(": ")", "{": "}", "[": "]"}


def _close(s, i):
    """Behind the bracket that opens at s[i]."""
    depth = 0
    for k in range(i, len(s)):
        depth += (s[k] in PAIR) - (s[k] in PAIR.values())
        if depth == 0:
            return k + 1
    return len(s)


def _to(s, i, stops):
    """The first of `stops` from s[i] on outside brackets, or the bracket that closes around s[i]."""
    while i < len(s) and s[i] not in stops and s[i] not in PAIR.values():
        i = _close(s, i) if s[i] in PAIR else i + 1
    return i


def _statement(s, i):
    """Behind the statement or block that begins at s[i], with its else."""
    i += len(s[i:]) - len(s[i:].lstrip())
    c = CONDITION.match(s, i)
    end = _statement(s, _close(s, c.end())) if c else _close(s, i) if s[i] == "{" else _to(s, i, ";") + 1
    other = re.compile(r"\s*else\b").match(s, end) if c else None
    return _statement(s, other.end()) if other else end


def _by_lane(text, names):
    """Where `text` first names a value that differs from lane to lane (-1: nowhere)."""
    for m in reversed(list(UNIFORM.finditer(text))):
        end = _close(text, m.end() - 1)
        text = text[:m.start()] + " " * (end - m.start()) + text[end:]
    at = [m.start() for m in re.finditer(r"\btid\(\)|\bthreadIdx\b", text)]
    at += [m.start() for n in names for m in re.finditer(r"(?<![\w.>])%s\b" % n, text)]
    return min(at, default=-1)


def lookups_by_lane(src):
    """(line, text) of the descriptor look-ups that are reached under a condition, or in a loop, whose terms differ from lane to lane."""
    src = re.sub(r"//[^\n]*", "", src)
    found = set()
    for f in re.finditer(r"^[^\s/#}][^;{}]*\)\s*\{", src, re.M):
        first, end = f.end() - 1, _close(src, f.end() - 1)
        body = src[first:end]
        decls = []                                           # name, value, where it is in scope
        for d in DECLARATION.finditer(body):
            stop = _to(body, d.end(), ";")
            block = _to(body, d.end(), "")
            block = _statement(body, block + 1) if body[block:block + 1] == ")" else block
            i = d.end()
            while i < stop:
                k = _to(body, i, ",;")
                m = NAME.match(body[i:k])
                if m and not re.match(r"\s*\[[&=]", m.group(2)):
                    decls.append((m.group(1), m.group(2), i, block))
                i = k + 1
        lane = set()
        while True:
            more = {d for d in decls if _by_lane(d[1], [n for n, _, a, b in lane if a <= d[2] < b]) >= 0} | lane
            if more == lane:
                break
            lane = more
        for c in CONDITION.finditer(body):
            past = _close(body, c.end())
            at = _by_lane(body[c.end():past], [n for n, _, a, b in lane if a <= c.end() < b or past > a >= c.end()])
            if at >= 0:
                for m in LOOKUP.finditer(body, c.end() + at, _statement(body, c.start())):
                    found.add((src.count("\n", 0, first + m.start()) + 1, src[first + m.start():].split("\n")[0][:60]))
    return sorted(found)


def test_descriptor_words_are_looked_up_with_all_lanes_on():
    """A descriptor is one register, a word per lane, and a look-up reads the lane of its word whether that is on or off.  A copy of the
    register that the compiler makes in a region for some lanes only holds the words of those, so no look-up lies in such a region."""
    with open(KERNELS) as f:
        assert lookups_by_lane(f.read()) == []


@pytest.mark.parametrize("code,lines", [
    ("if (tid() == 0) x = task[T_A0];", 1), ("if (task[HOT_TRACE] && tid() == 0) x = 1;", 0), ("if (tid() == 0 && task[HOT_TRACE]) x = 1;", 1),
    ("const int lane = tid() & 63, wave = sreg(tid() >> 6); if (wave == 0) x = op[O_K]; if (lane < 4) { y = 0; } else { x = op[O_K]; }", 1),
    ("for (int i = tid(); i < n; i += WG) { y[i] = store_buf(P, op); }", 1), ("for (int i = 0; i < n; ++i) x = op[O_K]; { const int i = tid(); y = i; }", 0),
    ("const int k = op[O_K]; for (int i = tid(); i < k; i += WG) y[i] = k;", 0)])
def test_the_rule_finds_what_it_names(code, lines):
    assert len(lookups_by_lane("void f() {\n" + code + "\n}\n")) == lines
