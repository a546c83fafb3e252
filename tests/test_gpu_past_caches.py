"""Outputs too large to stay in the last-level cache are written past it (optimizer's rounded copy, gradient of the logits,
weight gradients): the same bits as by the launches that do not."""
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2401_15207_amd", "csrc")


def line(name, source):
    """The size from which an output goes past the caches, as the source states it."""
    n, shift = re.search(r"%s = (?:int64_t\()?(\d+)\)?(?: << (\d+))?;" % name, open(os.path.join(CSRC, source)).read()).groups()
    return int(n) << int(shift or 0)


OPTS = {"adamw": dict(kind="adamw", eps=1e-8, momentum=0.0), "adagrad": dict(kind="adagrad", eps=1e-10, momentum=0.0),
        "sgdm": dict(kind="sgd", eps=1e-8, momentum=0.9), "sgd": dict(kind="sgd", eps=1e-8, momentum=0.0)}


@pytest.mark.gpu
@pytest.mark.parametrize("name", sorted(OPTS))
@pytest.mark.parametrize("n", [16000000, 150000000, 150000003])
def test_large_update_is_the_small_ones(name, n):
    import torch
    import paper_2401_15207_amd as H
    opt = dict(OPTS[name], lr=1e-3, beta1=0.9, beta2=0.999, weight_decay=0.01)
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    w, gr, s1 = (torch.randn(n, generator=g, device="cuda") * s for s in (0.02, 1e-3, 1e-4))
    s1 = s1.square() if name == "adagrad" else s1
    s2 = torch.rand(n, generator=g, device="cuda") * 1e-8
    s1, s2 = (None if name == "sgd" else s1), (s2 if name == "adamw" else None)
    # which product of AdamW's moments is fused follows from whether the count is a multiple of eight: the same for the parts as for the whole
    cut = n // 2 if n % 8 == 0 else 75000004
    at_line = line("OPT_FOUR_WAVES" if n < 100000000 else "OPT_COPY_PAST_CACHES", "elementwise.hip")  # (small launches keep more wavefronts)
    assert cut < at_line <= n
    half = torch.empty(n, device="cuda", dtype=torch.bfloat16)
    parts = [(t.clone() if t is not None else None) for t in (w, s1, s2)] + [torch.empty_like(half)]
    H.kernel_optimizer(opt, n, True, 3, w, gr, s1, s2, half)
    for a, b in ((0, cut), (cut, n)):
        at = [None if t is None else t[a:b] for t in parts]
        H.kernel_optimizer(opt, b - a, True, 3, at[0], gr[a:b], at[1], at[2], at[3])
    torch.cuda.synchronize()
    for x, y in zip((w, s1, s2, half), parts):
        assert x is None or torch.equal(x, y)
    assert torch.equal(half, w.to(torch.bfloat16))


@pytest.mark.gpu
@pytest.mark.parametrize("rows,vocab,dtype", [(1900, 32000, "bf16"), (1200, 50272, "bf16"), (1900, 16000, "fp32"), (1000, 30000, "fp32"), (4900, 12000, "bf16")])
def test_large_logits_are_the_small_ones(rows, vocab, dtype):
    """The second half of the rows has no target: the first half's gradient and the loss are those of a call of half the rows.  Both register kernels
    of either type, and rows that count their targets apart."""
    import torch
    import paper_2401_15207_amd as H
    dt, code = (torch.bfloat16, 1) if dtype == "bf16" else (torch.float32, 0)
    size = rows * vocab * dt.itemsize
    assert size // 2 < line("CE_PAST_CACHES_BYTES", "elementwise.hip") <= size
    g = torch.Generator(device="cuda")
    g.manual_seed(rows + vocab)
    big = (torch.randn(rows, vocab, generator=g, device="cuda") * 2.0).to(dt)
    labels = torch.randint(0, vocab, (rows,), generator=g, device="cuda", dtype=torch.int32)
    labels[rows // 2:] = -1
    small = big[:rows // 2].clone()
    losses = []
    for x, n in ((big, rows), (small, rows // 2)):
        losses.append(torch.empty(1, device="cuda"))
        H.kernel_cross_entropy(code, n, vocab, x, labels, torch.empty(n + 1, device="cuda"), losses[-1])
    torch.cuda.synchronize()
    assert torch.equal(big[:rows // 2], small) and not big[rows // 2:].any()
    assert torch.equal(*losses)


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K,cut", [(6144, 4096, 64, 3072), (6152, 4104, 40, 3072), (25176, 1000, 232, 12800), (256, 98400, 24, 128)])
def test_large_weight_gradient_is_the_small_ones(M, N, K, cut):
    """fp32 outputs of gemm_tt_k (whole tiles) and gemm_lds_k, in rows of a wider buffer, against two calls of half the rows each."""
    import torch
    import paper_2401_15207_amd as H
    g = torch.Generator(device="cuda")
    g.manual_seed(M + N + K)
    a, b = (torch.randn(K, n, generator=g, device="cuda").to(torch.bfloat16) for n in (M, N))
    whole, parts = (torch.full((M + 1, N + 8), 7.0, device="cuda") for _ in range(2))
    H.kernel_gemm(1, 0, 0, 1, M, N, K, a, M, b, N, whole, N + 8)
    for lo, hi in ((0, cut), (cut, M)):
        H.kernel_gemm(1, 0, 0, 1, hi - lo, N, K, a[:, lo:], M, b, N, parts[lo:], N + 8)
    torch.cuda.synchronize()
    assert torch.equal(whole, parts)
    assert (whole[M] == 7.0).all() and (whole[:, N:] == 7.0).all() and not (whole[:M, :N] == 7.0).all(1).any()
