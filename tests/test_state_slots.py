"""Which groups' state the device slots hold (csrc/state_slots.h): host bookkeeping, no GPU.  Random fetches and updates, with a
model of the slots' memory beside them: nothing kept is overwritten, and whatever is overwritten is either named as emptied (the
copy then waits for its write-back) or was emptied, and waited for, by an earlier copy on the same stream."""
import ctypes
import os
import random
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2401_15207_amd", "csrc")
SRC = r"""
#include "state_slots.h"
using hift::StateSlots;
static StateSlots s;
extern "C" void reset(int groups, int64_t cap) { s.reset(groups, cap); }
extern "C" int put(int g, int64_t floats, int spare, int* emptied) {
  std::vector<int> v;
  if (!s.put(g, floats, spare, v)) return -1;
  for (size_t i = 0; i < v.size(); ++i) emptied[i] = v[i];
  return (int)v.size();
}
extern "C" int slot(int g) { return s.slot(g); }
extern "C" int64_t at(int g) { return s.at(g); }
extern "C" int kept(int g) { return s.kept(g); }
extern "C" int recent(int g) { return s.recent(g); }
extern "C" int last() { return s.last(); }
extern "C" void keep(int g) { s.keep(g); }
extern "C" void let_go() { s.let_go(); }
extern "C" void updated(int g) { s.updated(g); }
"""


@pytest.fixture(scope="module")
def slots(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("clang++")
    if cxx is None:
        pytest.skip("needs a C++ compiler")
    d = tmp_path_factory.mktemp("state_slots")
    (d / "t.cpp").write_text(SRC)
    subprocess.run([cxx, "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, str(d / "t.cpp"), "-o", str(d / "t.so")], check=True)
    lib = ctypes.CDLL(str(d / "t.so"))
    lib.at.restype = ctypes.c_int64
    lib.put.argtypes = [ctypes.c_int, ctypes.c_int64, ctypes.c_int, ctypes.POINTER(ctypes.c_int)]
    lib.reset.argtypes = [ctypes.c_int, ctypes.c_int64]
    return lib


@pytest.mark.parametrize("groups", [1, 2, 3, 4, 5, 14, 34])
@pytest.mark.parametrize("sizes", ["alike", "mixed", "one_large"])
def test_a_place_is_given_up_only_where_the_copy_waits_for_it(slots, groups, sizes):
    rng = random.Random(groups)
    size = [{"alike": 1000, "mixed": rng.randint(1, 1000), "one_large": 1000 if g == 0 else rng.randint(60, 180)}[sizes] for g in range(groups)]
    cap = (max(size) + 63) // 64 * 64
    slots.reset(groups, cap)
    buf = (ctypes.c_int * groups)()
    live = {}  # group -> (slot, first, end): what a write-back may still read
    held_most = 0
    for _ in range(3000):
        g = rng.randrange(groups)
        if slots.slot(g) >= 0 and rng.random() < 0.5:
            slots.keep(g)
            slots.updated(g)
            assert slots.last() == g and slots.recent(g) and not slots.kept(g)
            continue
        if rng.random() < 0.05:
            slots.let_go()
        before = {o: (slots.slot(o), slots.at(o)) for o in range(groups) if slots.slot(o) >= 0}
        kept = {o for o in before if slots.kept(o)}
        spare = slots.last() if rng.random() < 0.5 else -1
        n = slots.put(g, size[g], spare, buf)
        if n < 0:
            assert all(slots.slot(o) == q and slots.at(o) == a for o, (q, a) in before.items())
            full = {q for o, (q, _a) in before.items() if o != g and (o in kept or o == spare)}
            assert len(full) == 3
            continue
        emptied = set(buf[:n])
        q, first = slots.slot(g), slots.at(g)
        assert first % 64 == 0 and first + size[g] <= cap and slots.kept(g)
        assert not emptied & kept and spare not in emptied and g not in emptied
        for o in emptied | {g}:
            live.pop(o, None)
        for o, (p, a, b) in live.items():
            assert p != q or first + size[g] <= a or b <= first, (g, o)
        live[g] = (q, first, first + size[g])
        assert {o for o in range(groups) if slots.slot(o) >= 0} == set(live)
        held_most = max(held_most, len(live))
    assert held_most >= min(groups, 3)


def test_a_kept_group_leaves_room_for_another_whatever_the_sizes(slots):
    """The one being updated never keeps the next from its place."""
    rng = random.Random(1)
    for _ in range(200):
        size = [rng.randint(1, 1000) for _ in range(9)]
        slots.reset(9, (max(size) + 63) // 64 * 64)
        buf = (ctypes.c_int * 9)()
        for t in range(60):
            cur = t % 9
            slots.let_go()
            if slots.slot(cur) >= 0:
                slots.keep(cur)
            else:
                assert slots.put(cur, size[cur], -1, buf) >= 0
            assert slots.put((cur + 1) % 9, size[(cur + 1) % 9], -1, buf) >= 0 and slots.slot(cur) >= 0
            slots.updated(cur)
