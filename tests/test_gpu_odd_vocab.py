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


# rows kept in registers in 16 and 32 pieces a thread, each also with gradients past the caches, with targets counted apart (more than 2048 rows), and
# rows too wide for registers
@pytest.mark.parametrize("rows,vocab", [(2048, 12466), (300, 50257), (64, 65541), (1216, 50257), (1920, 32003), (2560, 32003)])
def test_wide_odd_vocabulary_head(rows, vocab, monkeypatch):
    """Loss and head gradient against torch in 64 bits, from a model whose layer adds nothing to the embeddings, in memory that held NaN before: what
    follows a row of logits must have no part in either."""
    import torch
    import paper_2401_15207_amd as H
    seq, d, lr = 64 if rows % 64 == 0 else 60, 128, 1024.0
    cfg = dict(arch=2, n_layers=1, d_model=d, n_heads=2, d_ffn=256, vocab=vocab, max_seq=64, n_classes=0, norm_eps=1e-5, rope_base=10000.0, dtype=1)
    opt = dict(kind="sgd", lr=lr, beta1=0.0, beta2=0.0, eps=0.0, weight_decay=0.0, momentum=0.0)
    empty = torch.empty
    with monkeypatch.context() as mp:  # the model's arena
        mp.setattr(torch, "empty", lambda *a, **k: empty(*a, **k).fill_(255) if k.get("dtype") is torch.uint8 else empty(*a, **k))
        m = H.HiftModel(cfg, opt, 1, rows // seq, seq)
    g = torch.Generator(device="cuda")
    g.manual_seed(vocab)
    units, named = {}, {}
    for name, shape, kind, unit, _off in m.tensors:
        n = 1
        for s in shape:
            n *= s
        scale = 0.0 if name in ("l0.wo", "l0.wd") else 0.18 if name == "whead" else 1.0 if name == "tok_emb" else 0.02
        w = torch.randn(n, generator=g, device="cuda") * scale if kind != 1 else torch.ones(n, device="cuda")
        named[name] = w.to(torch.bfloat16).view(*shape)
        units.setdefault(unit, []).append(named[name].float().flatten())
    for u in units:
        m.write_params_device(u, u + 1, torch.cat(units[u]))
    k = m.set_group_schedule("bottom2up", 1, 0)
    tok = torch.randint(0, vocab, (rows // seq, seq), generator=g, device="cuda", dtype=torch.int32)
    lab = torch.full_like(tok, -1)
    lab[:, :-1] = torch.randint(0, vocab, (rows // seq, seq - 1), generator=g, device="cuda", dtype=torch.int32)
    lab[0, 0], lab[-1, 0] = vocab - 1, vocab - 2  # targets beside the end of the row
    before = torch.from_numpy(m.read_params(k - 1, k)).cuda()
    loss = m.step(tok, lab, k - 1)
    head = ((before - torch.from_numpy(m.read_params(k - 1, k)).cuda()) / lr)[-vocab * d:].view(vocab, d).double()  # after the last normalisation's gain

    x = named["tok_emb"][tok.flatten().long()].double()
    xf = (x / torch.sqrt((x * x).mean(1, keepdim=True) + 1e-5)).to(torch.bfloat16).double()
    logits = (xf @ named["whead"].double().T).to(torch.bfloat16).double()
    at = (lab.flatten() >= 0).nonzero()[:, 0]
    target = lab.flatten()[at].long()
    lse = torch.logsumexp(logits, 1)
    want = (lse[at] - logits[at, target]).mean()
    # a rounding of a logit that falls the other way moves its row's loss by 2^-8 of the logit at most, few of which do
    assert abs(loss - want.item()) <= 1e-4 * want.item()
    dl = torch.zeros_like(logits)
    dl[at] = torch.exp(logits[at] - lse[at, None])
    dl[at, target] -= 1.0
    ref = (dl / len(at)).T @ xf
    # each value of the logits' gradient is rounded to bf16 once: 2^-9 of it
    assert (head - ref).norm() <= 2.0 ** -8 * ref.norm()
    assert ((head - ref)[-8:].norm(dim=1) <= 2.0 ** -7 * ref[-8:].norm(dim=1)).all()  # (sums of few values: twice that)
    # each row of the logits' gradient sums to zero, so the rows of the head's gradient do, but for rounding
    assert head.sum(0).abs().max() <= 0.02 * head.abs().sum(0).max()
    assert torch.isfinite(head).all() and (head != 0).any(1).all()
