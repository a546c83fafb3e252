"""How a copy of optimizer state is split into the rectangles handed to the runtime (csrc/copy_parts.h): host arithmetic, no GPU.
A group's state may be many GB; a rectangle's pitch may not reach 2^31 bytes."""
import ctypes
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2401_15207_amd", "csrc")
SRC = r"""
#include "copy_parts.h"
// 0: the parts cover [0, bytes) in order without gap or overlap, and none is too long; otherwise the number of the rule broken
extern "C" int check(size_t bytes, size_t* n_rect, size_t* n_plain, size_t* widest, size_t* longest_plain) {
  size_t next = 0;
  *n_rect = *n_plain = *widest = *longest_plain = 0;
  const int e = hift::copy_parts(bytes, [&](size_t at, size_t row, size_t n) {
    if (at != next || n == 0 || n > bytes - at) return 1;
    if (row && n != 2 * row) return 2;
    if (row && row % 16 != 0) return 3;
    if (row && at % 32 != 0) return 4;
    next = at + n;
    size_t* count = row ? n_rect : n_plain;
    size_t* most = row ? widest : longest_plain;
    ++*count;
    if ((row ? row : n) > *most) *most = row ? row : n;
    return 0;
  });
  return e ? e : (next == bytes ? 0 : 5);
}
extern "C" int stops_at(size_t bytes, int part) {
  int seen = 0;
  const int e = hift::copy_parts(bytes, [&](size_t, size_t, size_t) { return ++seen == part ? 7 : 0; });
  return e == 7 && seen == part;
}
extern "C" size_t part_max() { return hift::COPY_PART_MAX; }
extern "C" size_t rect_min() { return hift::COPY_RECT_MIN; }
"""


@pytest.fixture(scope="module")
def parts(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("clang++")
    if cxx is None:
        pytest.skip("needs a C++ compiler")
    d = tmp_path_factory.mktemp("copy_parts")
    (d / "t.cpp").write_text(SRC)
    subprocess.run([cxx, "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, str(d / "t.cpp"), "-o", str(d / "t.so")], check=True)
    lib = ctypes.CDLL(str(d / "t.so"))
    lib.part_max.restype = lib.rect_min.restype = ctypes.c_size_t
    lib.check.argtypes = [ctypes.c_size_t] + [ctypes.POINTER(ctypes.c_size_t)] * 4
    lib.stops_at.argtypes = [ctypes.c_size_t, ctypes.c_int]
    return lib


def test_parts_cover_every_size_and_no_row_is_too_wide(parts):
    top, low = parts.part_max(), parts.rect_min()
    sizes = {0, 4, 16, 28, 32, 36, low - 4, low, low + 4, low + 28, low + 32, top - 4, top, top + 4, top + 28, top + low - 4,
             top + low + 20, 3 * top + 12}
    for gb in (2, 4, 10, 16):   # groups of several layers of the 7B and 13B shapes; 2^31 and 2^32 from both sides
        sizes |= {(gb << 30) + o for o in (-32, -4, 0, 4, 32, 780_000_004)}
    sizes |= {2 * 317_204_480 * 4 * m for m in (1, 2, 4)}  # one to four layers of width 5120, two state arrays
    for n in sizes:
        out = [ctypes.c_size_t() for _ in range(4)]
        assert parts.check(n, *map(ctypes.byref, out)) == 0, n
        n_rect, n_plain, widest, longest_plain = (x.value for x in out)
        assert widest <= top // 2 < 2 ** 31 - 1, n
        assert longest_plain < low and n_plain <= 1, n
        assert n_rect == n // top + (1 if n % top >= low else 0), n


def test_an_error_ends_the_copy(parts):
    top = parts.part_max()
    assert parts.stops_at(5 * top, 1) and parts.stops_at(5 * top, 3)
