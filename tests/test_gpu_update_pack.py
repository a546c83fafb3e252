"""The update that writes the fragment-order copies itself (opt_pack_k): after it, a model computes what a model computes whose copies
were packed from the same master weights, bit for bit, in the forward pass (loss) and in the backward pass (the update of the lowest
group, whose gradient crosses every transposed copy)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

OPTS = [dict(kind="adamw", lr=1e-3, beta1=0.9, beta2=0.999, eps=1e-8, weight_decay=0.01, momentum=0.0),
        dict(kind="adagrad", lr=1e-3, beta1=0.9, beta2=0.999, eps=1e-10, weight_decay=0.0, momentum=0.0),
        dict(kind="sgd", lr=1e-2, beta1=0.9, beta2=0.999, eps=1e-8, weight_decay=0.01, momentum=0.9),
        dict(kind="sgd", lr=1e-2, beta1=0.9, beta2=0.999, eps=1e-8, weight_decay=0.0, momentum=0.0)]
SHAPES = {
    # both copies, gains folded into the forward copies (either block order), an output matrix whose last 32-row tile is a quarter full
    "rotary": (dict(arch=2, n_layers=1, d_model=4096, n_heads=32, d_ffn=3584, vocab=3400, max_seq=512, n_classes=0), 4),
    # matrices with one of the two copies, the last tile of a row a quarter full
    "gelu": (dict(arch=0, n_layers=2, d_model=832, n_heads=13, d_ffn=3328, vocab=5003, max_seq=512, n_classes=0), 8),
}


@pytest.mark.parametrize("opt", OPTS, ids=["adamw", "adagrad", "sgdm", "sgd"])
@pytest.mark.parametrize("shape,parked", [("rotary", 0), ("rotary", 1), ("gelu", 0)])
def test_copies_are_those_of_the_new_weights(shape, parked, opt):
    import torch
    import paper_2401_15207_amd as H
    cfg, batch = SHAPES[shape]
    cfg = dict(cfg, norm_eps=1e-5, rope_base=10000.0, dtype=1)
    seq, units = 512, cfg["n_layers"] + 2
    g = torch.Generator(device="cuda").manual_seed(5)
    tok = torch.randint(0, cfg["vocab"], (batch, seq), generator=g, device="cuda", dtype=torch.int32)
    lab = torch.roll(tok, -1, 1)

    def model():
        return H.HiftModel(cfg, opt, 1, batch, seq, state_on_host=parked)

    a, b = model(), model()
    try:
        for t in range(units):
            n = a.read_params(t, t + 1).size
            a.write_params_device(t, t + 1, torch.randn(n, generator=g, device="cuda") * 0.02 + (0.5 if n <= 4 * cfg["d_model"] else 0.0))
        for m in (a, b):
            m.set_group_schedule("bottom2up", 1, 0)
        for _ in range(2):  # the second round updates from a state that is not zero
            for t in range(1, units):
                a.step(tok, lab, t)
        for t in range(units):
            b.write_params_device(t, t + 1, torch.from_numpy(a.read_params(t, t + 1)).cuda())
        la, lb = a.step(tok, lab, 0), b.step(tok, lab, 0)
        assert np.float32(la).tobytes() == np.float32(lb).tobytes(), (la, lb)
        wa, wb = a.read_params(0, 1), b.read_params(0, 1)
        assert np.array_equal(wa, wb), np.abs(wa - wb).max()
    finally:
        a.close()
        b.close()
