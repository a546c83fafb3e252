"""The update that writes the fragment-order copies itself (opt_pack_k): after it, a model computes what a model computes whose copies
were packed from the same master weights, bit for bit, in the forward pass (loss) and in the backward pass (the update of the lowest
group, whose gradient crosses every transposed copy); and its weights and state are those of the plain update."""
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


@pytest.mark.parametrize("parked", [0, 1])
@pytest.mark.parametrize("opt", OPTS, ids=["adamw", "adagrad", "sgdm", "sgd"])
def test_new_weights_and_state_are_those_of_the_plain_update(opt, parked):
    """Twelve packed matrices in one group, more than one launch takes: new weights and state are, bit for bit, what the plain update
    makes of the same gradients, and nothing is packed after it.  The gradients: the momentum that SGD leaves after its first step."""
    import torch
    import paper_2401_15207_amd as H
    cfg = dict(arch=2, n_layers=3, d_model=1024, n_heads=8, d_ffn=2816, vocab=3400, max_seq=512, n_classes=0, norm_eps=1e-5, rope_base=10000.0, dtype=1)
    units, batch, seq, pack = 5, 32, 512, 5  # pack: the profile's category of re-packing
    g = torch.Generator(device="cuda").manual_seed(9)
    tok = torch.randint(0, cfg["vocab"], (batch, seq), generator=g, device="cuda", dtype=torch.int32)
    lab = torch.roll(tok, -1, 1)
    n_state = {"adamw": 2, "adagrad": 1}.get(opt["kind"], 1 if opt["momentum"] else 0)
    a = H.HiftModel(cfg, opt, units, batch, seq, state_on_host=parked)
    try:
        theta = torch.randn(a.n_params, generator=g, device="cuda") * 0.02
        state = [torch.zeros_like(theta) for _ in range(n_state)]
        a.write_params_device(0, units, theta)
        a.set_group_schedule("bottom2up", units, 0)
        a.profile_enable(True)
        assert a.memory()["device_packed"] > 3 * a.n_params  # two copies of nearly everything, two bytes each
        for t in (1, 2):
            b = H.HiftModel(cfg, dict(OPTS[2], weight_decay=0.0), units, batch, seq)
            b.write_params_device(0, units, theta)
            b.set_group_schedule("bottom2up", units, 0)
            b.step(tok, lab, 0)
            grad = torch.from_numpy(b.read_state(0, units, 0)).cuda()
            b.close()
            a.step(tok, lab, 0)
            for _name, shape, kind, _unit, off in a.tensors:
                n = int(np.prod(shape))
                parts = [x[off:off + n].clone() for x in (theta, grad, *state)]
                H.kernel_optimizer(opt, n, kind == 0, t, parts[0], parts[1], *(parts[2:] + [None, None])[:2])
                for x, part in zip((theta, *state), (parts[0], *parts[2:])):
                    x[off:off + n] = part
            assert np.array_equal(a.read_params(), theta.cpu().numpy()), t
            for j in range(n_state):
                assert np.array_equal(a.read_state(0, units, j), state[j].cpu().numpy()), (t, j)
        assert a.profile_read(pack)[0] == 0
    finally:
        a.close()
