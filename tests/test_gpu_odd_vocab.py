"""bf16 models whose vocabulary is no multiple of eight: rows of logits padded to whole 16-byte pieces, gradients of every group and the loss against
the oracle, also at a batch below the maxima, with a tied table and with rows without a target."""
import pytest

from tests.test_gpu_step_bf16 import _gradient_check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("arch,vocab,tied", [(0, 301, 0), (0, 1023, 0), (2, 333, 0), (2, 258, 0), (0, 999, 1), (2, 1001, 1), (0, 4, 0)])
def test_gradients_with_an_odd_vocabulary(arch, vocab, tied):
    wl = dict(arch=arch, n_layers=2, d_model=128, n_heads=2, d_ffn=512 if arch == 0 else 384, vocab=vocab, max_seq=64, n_classes=0, norm_eps=1e-5,
              rope_base=10000.0, dtype=1, batch=3, seq=40, m=1, strategy="bottom2up", opt=dict(kind="adamw", lr=1e-3, beta1=0.9, beta2=0.999,
                                                                                              eps=1e-8, weight_decay=0.0))
    over = dict(tie_embeddings=1) if tied else {}
    _gradient_check(wl, lambda k: range(k), test="odd vocabulary %d" % vocab, **over)
    _gradient_check(wl, lambda k: [k - 1], seed=6, batch=2, seq=33, test="odd vocabulary %d, smaller batch" % vocab, **over)


@pytest.mark.parametrize("rows,vocab", [(2048, 12466), (300, 50257), (64, 65541)])
def test_wide_odd_vocabulary_head(rows, vocab):
    """Wide heads, up to more columns than the register kernel of the cross-entropy takes: the loss of a uniform guess, and a head gradient that
    reaches every row and sums to zero."""
    import torch
    import paper_2401_15207_amd as H
    seq = 64 if rows % 64 == 0 else 60
    cfg = dict(arch=2, n_layers=1, d_model=128, n_heads=2, d_ffn=256, vocab=vocab, max_seq=64, n_classes=0, norm_eps=1e-5, rope_base=10000.0, dtype=1)
    opt = dict(kind="sgd", lr=1.0, beta1=0.0, beta2=0.0, eps=0.0, weight_decay=0.0, momentum=0.0)
    m = H.HiftModel(cfg, opt, 1, rows // seq, seq)
    g = torch.Generator(device="cuda")
    g.manual_seed(vocab)
    units = {}
    for name, shape, kind, unit, _off in m.tensors:
        n = 1
        for s in shape:
            n *= s
        w = torch.randn(n, generator=g, device="cuda") * 0.02 + (1.0 if kind == 1 else 0.0)
        units.setdefault(unit, []).append(w.to(torch.bfloat16).float())
    for u in units:
        m.write_params_device(u, u + 1, torch.cat(units[u]))
    k = m.set_group_schedule("bottom2up", 1, 0)
    tok = torch.randint(0, vocab, (rows // seq, seq), generator=g, device="cuda", dtype=torch.int32)
    lab = torch.full_like(tok, -1)
    lab[:, :-1] = tok[:, 1:]
    before = torch.from_numpy(m.read_params(k - 1, k)).cuda()
    loss = m.step(tok, lab, k - 1)
    assert abs(loss - torch.log(torch.tensor(float(vocab))).item()) < 0.2  # logits of nearly nothing: the loss of a uniform guess
    grad = before - torch.from_numpy(m.read_params(k - 1, k)).cuda()
    head = grad[-vocab * 128:].view(vocab, 128)  # after the last normalisation's gain
    # each row of the logits' gradient sums to zero, so the rows of the head's gradient do, but for rounding
    total = head.double().sum(0)
    assert total.abs().max() <= 0.02 * head.double().abs().sum(0).max()
    assert torch.isfinite(head).all() and (head != 0).any(1).all()
