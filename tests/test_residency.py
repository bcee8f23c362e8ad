"""CPU test of the rule that picks the 14-state kernel's form (csrc/residency.h): letting a launch
take the two-waves-per-SIMD form must not make a mix of launches wait for ever that found its
places with every launch at three waves per SIMD.

The model: a compute unit has four SIMDs of 512 registers per lane; a workgroup puts its waves on
them (1 wave of 168 or, in the two-waves form, 256 registers per SIMD for 16 knots, and the other
shapes' loads), and an XCD is a number of such units.  The parts of a problem wait for each other, so a
mix can wait for ever if some of its gangs can be placed so that each misses a part and no unit
has room for any missing one; the dispatch order is not known, so every filling counts.  A problem
of one part never waits."""
import ctypes
import functools
import itertools
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2309_08079_amd", "csrc")

# waves on each SIMD and registers per lane: 16 knots at two and at three waves per SIMD, 32 knots
# and 48 knots
SHAPES = {"two": ((1, 1, 1, 1), 256), "16": ((1, 1, 1, 1), 168), "32": ((2, 2, 2, 2), 256), "48": ((3, 3, 3, 3), 168)}


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    d = tmp_path_factory.mktemp("residency")
    src, lib = str(d / "rule.cpp"), str(d / "rule.so")
    with open(src, "w") as f:
        f.write('#include "residency.h"\nextern "C" int rule(int parts, long tasks, long places) '
                "{ return mpc::two_waves_form(parts, tasks, places); }\n")
    subprocess.run(["g++", "-shared", "-fPIC", "-std=c++17", "-I", CSRC, src, "-o", lib], check=True)
    f = ctypes.CDLL(lib).rule
    f.argtypes = [ctypes.c_int, ctypes.c_long, ctypes.c_long]
    return lambda parts, tasks, places: bool(f(parts, tasks, places))


def room(use, shape):
    waves, regs = SHAPES[shape]
    n = tuple(u + w * regs for u, w in zip(use, waves))
    return n if max(n) <= 512 else None


@functools.lru_cache(None)
def full_units(shapes):
    """workgroups of each shape on a compute unit that has room for none of the shapes"""
    todo, seen, full = [((0,) * len(shapes), (0, 0, 0, 0))], set(), set()
    while todo:
        count, use = todo.pop()
        if (count, use) in seen:
            continue
        seen.add((count, use))
        more = [(i, room(use, s)) for i, s in enumerate(shapes)]
        if not any(n for _, n in more):
            full.add(count)
        todo += [(count[:i] + (count[i] + 1,) + count[i + 1:], n) for i, n in more if n]
    return sorted(full)


@functools.lru_cache(None)
def waits_for_ever(gangs, units):
    gangs = tuple(g for g in gangs if g[1] > 1)
    for k in range(1, len(gangs) + 1):
        for some in set(itertools.combinations(gangs, k)):
            shapes = tuple(sorted({s for s, _ in some}))
            most = tuple(sum(p - 1 for s, p in some if s == t) for t in shapes)
            have = {(0,) * len(shapes)}
            for _ in range(units):
                sums = {tuple(a + b for a, b in zip(h, f)) for h in have for f in full_units(shapes)}
                have = {v for v in sums if all(x <= m for x, m in zip(v, most))}
            if have:
                return True
    return False


def taken(rule, gangs, units):
    return tuple(sorted(("two" if s == "16" and rule(p, p, 2 * units) else s, p) for s, p in gangs))


def test_model_on_plain_counts():
    assert not waits_for_ever((("16", 12),), 4) and waits_for_ever((("16", 13),), 4)
    assert not waits_for_ever((("two", 8),), 4) and waits_for_ever((("two", 9),), 4)
    assert not waits_for_ever((("48", 4),), 4) and waits_for_ever((("48", 3), ("48", 3)), 4)
    # 16, 16, 32 and 32 parts on the 32 units of an XCD
    assert not waits_for_ever((("16", 16), ("16", 16), ("16", 32), ("16", 32)), 32)
    assert waits_for_ever((("two", 16), ("two", 16), ("16", 32), ("16", 32)), 32)


@pytest.mark.parametrize("units", [2, 3, 4])
def test_no_mix_loses_its_places(rule, units):
    gangs = [("16", p) for p in range(1, 3 * units + 1)] + [(s, p) for s in ("32", "48") for p in range(2, units + 1)]
    for n in (1, 2, 3):
        for mix in itertools.combinations_with_replacement(gangs, n):
            mix = tuple(sorted(mix))
            if not waits_for_ever(mix, units):
                assert not waits_for_ever(taken(rule, mix, units), units), mix


@pytest.mark.parametrize("mix", [(32, 32, 16, 16), (32, 16, 16, 16), (80, 16), (94, 2), (32, 32, 27, 5), (48, 16, 16, 16),
                                 (16, 16, 16, 16, 16, 16)])
def test_mixes_that_fill_an_xcd(rule, mix):
    gangs = tuple(sorted(("16", p) for p in mix))
    assert not waits_for_ever(gangs, 32)
    assert not waits_for_ever(taken(rule, gangs, 32), 32)


def test_both_sides_of_the_line(rule):
    assert rule(1, 1, 1) and rule(1, 512, 512) and not rule(1, 513, 512)
    assert not rule(2, 2, 512) and not rule(16, 16, 64) and not rule(32, 512, 512)
