"""Contractions over long k that take one round of large tiles (csrc/lds_tiles.h, LDS_LONG_TILES): edges of the tiles and of the stages, in all
four layouts and both output types, with bias and residual and as several problems of a launch, against float64."""
import numpy as np
import pytest

from tests.lds_cases import LONG_BATCHES, LONG_CASES, LONG_EXTRAS
from tests.test_lds_tiles import lib  # noqa: F401 (fixture)


def test_the_cases_take_both_tiles_and_the_line_holds(lib):  # noqa: F811
    assert {lib.pick_long(*c, 1) for c in LONG_CASES} == {0, 1}
    # shorter k, more than one round, and few tiles keep the choice of lds_tile (measured: lds_tiles.h)
    for c in [(720, 4096, 1024), (720, 12288, 4096), (231, 4096, 22016), (231, 8192, 4096), (64, 32000, 4096)]:
        assert lib.pick_long(*c, 1) == -1


@pytest.mark.gpu
@pytest.mark.parametrize("ak,bk", [(1, 1), (1, 0), (0, 1), (0, 0)])
@pytest.mark.parametrize("M,N,K", LONG_CASES)
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


@pytest.mark.gpu
@pytest.mark.parametrize("ak,bk", [(1, 1), (1, 0), (0, 1), (0, 0)])
@pytest.mark.parametrize("M,N,K", LONG_EXTRAS)
def test_long_contraction_with_bias_and_residual(ak, bk, M, N, K):
    import torch
    import paper_2401_15207_amd as H
    g = torch.Generator(device="cuda")
    g.manual_seed(M + N + K + 2 * ak + bk + 1)
    a, b = (torch.randn(n, K, generator=g, device="cuda").to(torch.bfloat16) for n in (M, N))
    da, db = (x if kmajor else x.T.contiguous() for x, kmajor in ((a, ak), (b, bk)))
    bias = torch.randn(N, generator=g, device="cuda").to(torch.bfloat16)
    ref = a.double() @ b.double().T
    scale = K ** 0.5 + 1.0
    for out_f32 in (0, 1):
        dt = torch.float32 if out_f32 else torch.bfloat16
        res = torch.randn(M, N + 8, generator=g, device="cuda").to(dt)
        for with_bias, with_res in ((1, 0), (0, 1), (1, 1)):
            c = torch.full((M + 1, N + 8), 7.0, dtype=dt, device="cuda")
            H.kernel_gemm(1, ak, bk, out_f32, M, N, K, da, da.shape[1], db, db.shape[1], c, N + 8, bias if with_bias else None, res if with_res else None)
            want = ref + with_bias * bias.double() + with_res * res[:, :N].double()
            got = c.double()
            assert (got[M] == 7.0).all() and (got[:, N:] == 7.0).all()
            # as without them, plus a rounding of each sum to the output's type
            tol = 1e-5 * (want.abs() + scale) if out_f32 else 2 ** -8 * (want.abs() + ref.abs() + 0.02 * scale)
            assert ((got[:M, :N] - want).abs() <= tol).all(), (out_f32, with_bias, with_res)


@pytest.mark.gpu
@pytest.mark.parametrize("ak,bk", [(1, 1), (1, 0), (0, 1), (0, 0)])
@pytest.mark.parametrize("M,N,K,nz", LONG_BATCHES)
def test_long_contractions_of_a_batch(ak, bk, M, N, K, nz):
    import torch
    import paper_2401_15207_amd as H
    g = torch.Generator(device="cuda")
    g.manual_seed(M + N + K + 2 * ak + bk + 2)
    a, b = (torch.randn(nz, n, K, generator=g, device="cuda").to(torch.bfloat16) for n in (M, N))
    da, db = (x if kmajor else x.transpose(1, 2).contiguous() for x, kmajor in ((a, ak), (b, bk)))
    scale = K ** 0.5 + 1.0
    for out_f32 in (0, 1):
        c = torch.full((nz, M + 1, N + 8), 7.0, dtype=torch.float32 if out_f32 else torch.bfloat16, device="cuda")
        H.kernel_gemm(1, ak, bk, out_f32, M, N, K, da, da.shape[2], db, db.shape[2], c, N + 8, None, None, nz, M * K, N * K, (M + 1) * (N + 8))
        for z in range(nz):
            want, got = a[z].double() @ b[z].double().T, c[z].double()
            assert (got[M] == 7.0).all() and (got[:, N:] == 7.0).all()
            tol = 1e-5 * (want.abs() + scale) if out_f32 else 2 ** -8 * (want.abs() + 0.02 * scale)
            assert ((got[:M, :N] - want).abs() <= tol).all(), (out_f32, z)
