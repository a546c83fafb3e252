"""Contractions over long k that take one round of large tiles (csrc/lds_tiles.h, LDS_LONG_TILES): edges of the tiles and of the stages, in all
four layouts and both output types, against float64."""
import ctypes
import subprocess

import numpy as np
import pytest

from tests.test_lds_tiles import CSRC, SRC

# M, N, K: rows and columns that end inside a tile or fill it, k that ends inside a stage or fills it, the shortest k that qualifies
CASES = [(232, 11016, 4104), (720, 4096, 4096), (128, 24608, 3848), (1288, 3336, 1544), (256, 16520, 1536), (1024, 4096, 4160)]


@pytest.fixture(scope="module")
def pick(tmp_path_factory):
    d = tmp_path_factory.mktemp("lds_long")
    (d / "t.cpp").write_text(SRC + 'extern "C" int pick_long(int64_t M, int64_t N, int64_t K) { return hift::lds_long_tile(M, N, K, 1); }\n')
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, str(d / "t.cpp"), "-o", str(d / "t.so")], check=True)
    f = ctypes.CDLL(str(d / "t.so")).pick_long
    f.argtypes = [ctypes.c_int64] * 3
    return f


def test_the_cases_take_both_tiles_and_the_line_holds(pick):
    assert {pick(*c) for c in CASES} == {0, 1}
    # shorter k, more than one round, and few tiles keep the choice of lds_tile (measured: lds_tiles.h)
    for c in [(720, 4096, 1024), (720, 12288, 4096), (231, 4096, 22016), (231, 8192, 4096), (64, 32000, 4096)]:
        assert pick(*c) == -1


@pytest.mark.gpu
@pytest.mark.parametrize("ak,bk", [(1, 1), (1, 0), (0, 1), (0, 0)])
@pytest.mark.parametrize("M,N,K", CASES)
def test_long_contraction(ak, bk, M, N, K):
    import torch
    import paper_2401_15207_amd as H
    g = torch.Generator(device="cuda")
    g.manual_seed(M + N + K + 2 * ak + bk)

    def operand(rows, kmajor):  # inside a wider buffer of NaN: nothing beyond the operand's own rows and k may reach a result
        x = torch.randn(rows, K, generator=g, device="cuda").to(torch.bfloat16)
        t = x if kmajor else x.T
        wide = torch.full((t.shape[0] + 1, t.shape[1] + 8), float("nan"), dtype=torch.bfloat16, device="cuda")
        wide[:t.shape[0], :t.shape[1]] = t
        return x, wide
    (a, wa), (b, wb) = operand(M, ak), operand(N, bk)
    ref = (a.double() @ b.double().T).cpu().numpy()
    scale = np.sqrt(K) + 1.0
    for out_f32 in (0, 1):
        c = torch.full((M + 1, N + 8), 7.0, dtype=torch.float32 if out_f32 else torch.bfloat16, device="cuda")
        H.kernel_gemm(1, ak, bk, out_f32, M, N, K, wa, wa.shape[1], wb, wb.shape[1], c, N + 8)
        torch.cuda.synchronize()
        got = c.double().cpu().numpy()
        assert (got[M] == 7.0).all() and (got[:, N:] == 7.0).all()
        # fp32 sums of exact products, as in the other contraction tests; a bf16 result is rounded once
        tol = 1e-5 * (np.abs(ref) + scale) if out_f32 else 2 ** -8 * (np.abs(ref) + 0.02 * scale)
        assert (np.abs(got[:M, :N] - ref) <= tol).all()
