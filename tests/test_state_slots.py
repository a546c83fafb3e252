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
extern "C" int advance(int gid, const int* order, int k, int64_t t, const int64_t* floats, int* fetched, int* lost) {
  int n = 0;  // lost[g]: g's place was given up
  std::vector<int> v;
  s.advance(gid, std::vector<int32_t>(order, order + k), t, [&](int g, int spare, bool* done) {
    if ((*done = s.put(g, floats[g], spare, v))) fetched[n++] = g;
    for (int o : v) lost[o] = 1;
    return 0;
  });
  s.updated(gid);
  return n;
}
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
    lib.advance.argtypes = [ctypes.c_int, ctypes.c_void_p, ctypes.c_int, ctypes.c_int64, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p]
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


SIZES = {"embeddings": [1000] + [160] * 12 + [100], "deep": [1000] + [160] * 33, "alike": [160] * 34, "few": [160] * 5, "four": [160] * 4}
ORDERS = {"on": lambda i, rng: "next", "one in ten": lambda i, rng: "any" if rng.random() < 0.1 else "next",
          "every other": lambda i, rng: "any" if i % 2 else "next", "twice": lambda i, rng: "same" if i % 2 else "next", "any": lambda i, rng: "any"}


def one_group_to_a_slot(size, groups):
    """Values copied in where every slot holds one group and only the next of the schedule is fetched ahead."""
    held, at, k, copied = [-1] * 3, 0, len(size), 0
    for t, g in enumerate(groups):
        if g in held:
            at = held.index(g)
        else:
            held[at] = g
            copied += size[g]
        following = (t + 1) % k
        if g == t % k and following not in held:
            held[(at + 1) % 3] = following
            copied += size[following]
        at = (at + 1) % 3
    return copied


@pytest.mark.parametrize("sizes", SIZES)
@pytest.mark.parametrize("visits", ORDERS)
def test_steps_off_the_schedule_do_not_copy_the_same_state_again(slots, sizes, visits):
    """Groups in the schedule's order, in another one, and mixed: a step queues its own group, if need be, and at most two more;
    nothing is copied again that a slot still holds unused; and in all hardly more than with one group to a slot (where there are
    hardly more groups than slots, which one is given up is luck: up to half more)."""
    size, rng = SIZES[sizes], random.Random(7)
    k = len(size)
    order, floats, buf = (ctypes.c_int * k)(*range(k)), (ctypes.c_int64 * k)(*size), (ctypes.c_int * (2 * k))()
    slots.reset(k, (max(size) + 63) // 64 * 64)
    groups, fresh, copied = [], set(), 0  # fresh: copied in and not updated since
    for t in range(40 * k):
        kind = ORDERS[visits](t, rng)
        g = t % k if kind == "next" else groups[-1] if kind == "same" else rng.randrange(k)
        lost = (ctypes.c_int * k)()
        fetched = buf[:slots.advance(g, order, k, t, floats, buf, lost)]
        assert slots.slot(g) >= 0 and (g == t % k or set(fetched) <= {g}) and len([o for o in fetched if o != g]) <= 2
        fresh -= {o for o in range(k) if lost[o]}
        assert not set(fetched) & fresh, (t, g, fetched)
        copied += sum(size[o] for o in fetched)
        fresh = (fresh | {o for o in fetched if slots.slot(o) >= 0}) - {g}
        groups.append(g)
    plain, updated = one_group_to_a_slot(size, groups), sum(size[g] for g in groups)
    if visits == "on":
        assert copied - updated <= 3 * max(size)  # what is fetched ahead at the end
    assert copied <= (1.5 if k <= 5 else 1.1) * plain + 3 * max(size)
