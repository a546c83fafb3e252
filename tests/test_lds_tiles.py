"""Which tile of gemm_lds_k a contraction gets (csrc/lds_tiles.h): host arithmetic, no GPU."""
import ctypes
import os
import shutil
import subprocess

import pytest

from tests.lds_cases import LONG_BATCHES, LONG_CASES, LONG_EXTRAS
from tests.test_gpu_kernels import LDS_CASES
from tests.test_gpu_step_bf16 import GELU_CASES

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2401_15207_amd", "csrc")
SRC = r"""
#include "lds_tiles.h"
extern "C" int pick_long(int64_t M, int64_t N, int64_t K, int64_t nz) { return hift::lds_long_tile(M, N, K, nz); }
// what a contraction without a band gets: a tile for long k (after the others in tile()'s numbers) where one applies, else lds_tile's
extern "C" int pick(int64_t M, int64_t N, int64_t K, int64_t nz) {
  const int l = hift::lds_long_tile(M, N, K, nz);
  return l < 0 ? hift::lds_tile(M, N, K, nz) : hift::N_LDS_TILES + l;
}
extern "C" int tile(int i, int* bm, int* bn) {
  if (i >= hift::N_LDS_TILES + hift::N_LDS_LONG_TILES) return 0;
  const hift::LdsTile& t = i < hift::N_LDS_TILES ? hift::LDS_TILES[i] : hift::LDS_LONG_TILES[i - hift::N_LDS_TILES];
  *bm = t.bm;
  *bn = t.bn;
  return 1;
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("clang++")
    if cxx is None:
        pytest.skip("needs a C++ compiler")
    d = tmp_path_factory.mktemp("lds_tiles")
    (d / "t.cpp").write_text(SRC)
    subprocess.run([cxx, "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, str(d / "t.cpp"), "-o", str(d / "t.so")], check=True)
    lib = ctypes.CDLL(str(d / "t.so"))
    lib.pick.argtypes = lib.pick_long.argtypes = [ctypes.c_int64] * 4
    return lib


def tiles(lib):
    out, bm, bn = [], ctypes.c_int(), ctypes.c_int()
    while lib.tile(len(out), ctypes.byref(bm), ctypes.byref(bn)):
        out.append((bm.value, bn.value))
    return out


def test_the_gpu_cases_reach_every_tile(lib):
    """With rows and columns that end inside a tile and stages that end inside 64 k."""
    t = tiles(lib)
    cases = LDS_CASES + LONG_CASES
    reached = {lib.pick(M, N, K, 1) for M, N, K in cases if M % 64 and N % 64 and K % 64}
    assert reached >= set(range(len(t))) - {i for i, x in enumerate(t) if x == (64, 64)}
    assert {lib.pick(*c, 1) for c in cases} == set(range(len(t)))
    assert {lib.pick(batch * seq, f, d, 1) for _arch, batch, seq, d, f in GELU_CASES} == set(range(len(t)))
    # bias, residual and several problems in a launch, on the tiles for long k
    long_ones = set(range(len(t) - 2, len(t)))
    assert {lib.pick(*c, 1) for c in LONG_EXTRAS} == long_ones and {lib.pick(*c) for c in LONG_BATCHES} == long_ones


# problem, tile; beside it the time that was measured on this tile and on another, microseconds
MEASURED = [
    ((128, 64, 128, 512), (128, 64)),       # 7.5, 64 x 64: 9.2
    ((512, 512, 128, 128), (128, 128)),     # 32.6, 64 x 64: 37.2
    ((64, 64, 128, 2048), (64, 64)),        # 15.5, 128 x 64: 19.1
    ((1024, 1024, 64, 32), (128, 128)),     # 23.3, 64 x 64: 27.2
    ((231, 4096, 11008, 1), (64, 64)),      # 39.5, 128 x 64: 57.4
    ((2048, 4096, 1024, 1), (128, 128)),    # 24.1, 256 x 256: 28.0
    ((2048, 32000, 4096, 1), (256, 256)),   # 442, 128 x 128: 594
    ((8192, 4096, 11008, 1), (256, 256)),   # 556, 128 x 128: 753
    ((256, 51200, 1024, 1), (256, 256)),    # 32.0, 128 x 128: 40.0
    ((2048, 4096, 4096, 1), (256, 128)),    # (ring of three) 67, 128 x 128: 77
    ((16384, 16384, 256, 1), (128, 128)),   # 246, 256 x 256: 275
]


@pytest.mark.parametrize("problem,tile", MEASURED)
def test_measured_choices(lib, problem, tile):
    assert tiles(lib)[lib.pick(*problem)] == tile
