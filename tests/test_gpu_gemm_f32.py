"""The contraction of fp32 operands and of bf16 ones outside 16-byte pieces (csrc/gemm_f32.hip): every output is one chain of
fused multiply-adds over ascending k, so it is compared bit for bit with that chain, formed in 80-bit floating point and rounded
to 32 bits after every product (a product of two fp32 values and a third one need more than the 64 bits of that mantissa only
where the smaller of the two summands lies 2^-40 below the larger, far below the rounding that follows)."""
import itertools

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# tiles of 32 and 64, passes of 16 (64 x 64 tiles only), 32, 64, 128 and 256 k, fours and sixteens of k
SMALL = [(1, 1, 1), (31, 33, 3), (33, 31, 63), (64, 64, 64), (17, 65, 65), (65, 16, 128), (40, 9, 129), (64, 64, 256), (33, 34, 257), (5, 70, 530)]
LARGE = [(1024, 1024, 16), (1023, 1025, 5), (1025, 1000, 33), (1024, 1024, 65)]


def chain(a, b):
    """a [M, K], b [N, K]"""
    acc = np.zeros((a.shape[0], b.shape[0]), dtype=np.float32)
    for k in range(a.shape[1]):
        acc = (a[:, k, None].astype(np.longdouble) * b[None, :, k].astype(np.longdouble) + acc).astype(np.float32)
    return acc


@pytest.mark.parametrize("M,N,K", SMALL + LARGE)
@pytest.mark.parametrize("bf16", [0, 1])
def test_every_output_is_one_chain_over_ascending_k(M, N, K, bf16):
    import torch

    import paper_2401_15207_amd as H
    assert np.finfo(np.longdouble).nmant >= 63
    g = torch.Generator().manual_seed(M * 7 + N * 3 + K)
    dt = torch.bfloat16 if bf16 else torch.float32
    scale = torch.exp2(torch.randint(-6, 7, (1, K), generator=g).float())
    a, b = ((torch.randn(r, K, generator=g) * scale).to(dt) for r in (M, N))
    want = chain(a.float().numpy(), b.float().numpy())
    layouts = list(itertools.product((1, 0), (1, 0))) if M * N < 1 << 18 else [(1, 1), (0, 0)]
    for i, (ak, bk) in enumerate(layouts):
        pad = (1, 0, 3, 4)[i]   # bf16: odd leading dimensions keep the 16-byte kernel away; C with and without whole fours
        A, B = (torch.nn.functional.pad(t if km else t.T, (0, 1 | pad if bf16 else pad)).contiguous().cuda() for t, km in ((a, ak), (b, bk)))
        C = torch.full((M, N + pad), 7.0, device="cuda")
        H.kernel_gemm(bf16, ak, bk, 1, M, N, K, A, A.shape[1], B, B.shape[1], C, C.shape[1])
        got = C.cpu().numpy()
        assert np.array_equal(got[:, :N], want), (ak, bk)
        assert (got[:, N:] == 7.0).all()


def test_bias_residual_and_batches():
    import torch

    import paper_2401_15207_amd as H
    rng = np.random.default_rng(3)
    for batch, (M, N, K) in itertools.product((1, 3), [(33, 36, 70), (31, 35, 20)]):
        a, b = (rng.standard_normal((batch, r, K)).astype(np.float32) for r in (M, N))
        r = rng.standard_normal((batch, M, N)).astype(np.float32)
        bias = rng.standard_normal(N).astype(np.float32)
        A, B, R, BI = (torch.from_numpy(x).cuda() for x in (a, b, r, bias))
        C = torch.empty_like(R)
        H.kernel_gemm(0, 1, 1, 0, M, N, K, A, K, B, K, C, N, BI, R, batch=batch, sa=M * K, sb=N * K, sc=M * N)
        want = np.stack([(chain(a[z], b[z]) + bias) + r[z] for z in range(batch)])
        assert np.array_equal(C.cpu().numpy(), want)


def test_rows_too_far_apart_for_32_bit_offsets():
    import torch

    import paper_2401_15207_amd as H
    rng = np.random.default_rng(5)
    for M, N, K, ak, bk, lda, ldb in [(35, 3, 71, 1, 1, 71, 8_400_000), (35, 3, 71, 1, 0, 71, 2_100_000), (35, 3, 71, 0, 1, 2_100_000, 71),
                                      (35, 3, 71, 0, 0, 35, 2_100_000), (1000, 1030, 13, 0, 1, 2_100_000, 13), (1030, 1000, 16, 1, 0, 16, 2_100_000)]:
        a, b = (rng.standard_normal((r, K)).astype(np.float32) for r in (M, N))
        want = chain(a, b)
        A = torch.zeros(M if ak else K, lda, device="cuda")
        B = torch.zeros(N if bk else K, ldb, device="cuda")
        A[:, :K if ak else M] = torch.from_numpy(a if ak else a.T.copy()).cuda()
        B[:, :K if bk else N] = torch.from_numpy(b if bk else b.T.copy()).cuda()
        C = torch.empty(M, N, device="cuda")
        H.kernel_gemm(0, ak, bk, 0, M, N, K, A, lda, B, ldb, C, N)
        assert np.array_equal(C.cpu().numpy(), want), (ak, bk)
