"""fp32 models through the fused attention (csrc/attention_f32.hip), GELU on the way out of a contraction and the column sums in one
launch: gradients of every group (plain SGD at rate 1) against the float64 oracle at the edges of the kernels' ranges, and against
the separate kernels where those give the same bits."""
import numpy as np
import pytest

from hift_inputs import WORKLOADS, make_batch, model_config
from tests.hift_pair import initial_weights, make_pair, to_dev

pytestmark = pytest.mark.gpu

SGD1 = dict(kind="sgd", lr=1.0, beta1=0, beta2=0, eps=0, weight_decay=0.0, momentum=0.0)
TOL = 1e-5  # fp32 sums; the bar of the fp32 steps


def _compare_gradients(wl, seed):
    """Every group's step from the same weights: the gradient as a whole, and that of gains and biases."""
    orc, gpu, theta0 = make_pair(wl, seed=seed, jitter=0.05)
    for t in range(1, orc.k + 1):
        gid = orc.schedule_group_at(t)
        orc.theta[:] = theta0
        gpu.write_params(0, gpu.n_units, theta0)
        tok, lab = make_batch(wl, seed, t)
        want_loss, loss = orc.step(tok, lab, gid), gpu.step(*to_dev(tok, lab), gid)
        assert abs(loss - want_loss) <= TOL * max(abs(want_loss), 1.0), (t, want_loss, loss)
        got, want = gpu.read_params() - np.asarray(theta0, np.float64), orc.theta - theta0
        # a weight that moved is rounded to 2^-24 of itself, which the difference of two weights shows
        moved, rounding = want != 0, 2.0 ** -24 * np.abs(theta0)
        assert np.linalg.norm(got - want) <= TOL * np.linalg.norm(want) + np.linalg.norm(rounding[moved]), t
        ones = np.zeros(got.size, bool)
        for _name, shape, _kind, _unit, off in gpu.tensors:
            if len(shape) == 1:
                ones[off:off + shape[0]] = True
        assert np.linalg.norm((got - want)[ones]) <= TOL * np.linalg.norm(want[ones]) + np.linalg.norm(rounding[ones & moved]), t


# sixteens of queries and keys, powers of two of them (32, 64; longer sequences take separate kernels), heads of less than, one, two and four
# sixteens
@pytest.mark.parametrize("arch,batch,seq,heads,hd", [
    (0, 2, 1, 2, 16), (1, 3, 5, 2, 4), (0, 1, 16, 3, 16), (1, 2, 17, 3, 20), (2, 2, 32, 2, 32), (0, 2, 33, 2, 32), (1, 1, 64, 2, 36), (2, 1, 65, 2, 64),
    (0, 1, 127, 2, 48), (1, 1, 128, 1, 64), (0, 2, 129, 2, 16), (1, 1, 250, 2, 64), (2, 1, 256, 2, 64), (0, 1, 257, 2, 16), (0, 2, 24, 2, 68)])
def test_gradients_at_the_edges(arch, batch, seq, heads, hd):
    d = heads * hd
    wl = dict(arch=arch, n_layers=1, d_model=d, n_heads=heads, d_ffn=2 * d, vocab=64, max_seq=max(seq, 8), n_classes=2 if arch == 1 else 0, norm_eps=1e-5,
              rope_base=10000.0, dtype=0, batch=batch, seq=seq, m=1, strategy="top2down", opt=SGD1)
    _compare_gradients(wl, 41)


def _grads(wl, unfused, seq):
    import paper_2401_15207_amd as H
    theta0 = initial_weights(model_config(wl), 43, 0.05)
    gpu = H.HiftModel(model_config(wl), SGD1, 1, wl["batch"], seq, init_params=theta0, unfused=unfused)
    k = gpu.set_group_schedule("top2down", 1)
    losses = [gpu.step(*to_dev(*make_batch(dict(wl, seq=seq), 43, t)), gpu.schedule_group_at(t)) for t in range(1, k + 1)]
    return np.array(losses), gpu.read_params()


@pytest.mark.parametrize("seq,hd", [(1, 16), (3, 4), (16, 20), (31, 16), (32, 32), (47, 32), (64, 48), (65, 64), (100, 16), (128, 20), (131, 64),
                                    (192, 16), (193, 32), (256, 64)])
@pytest.mark.parametrize("arch", [0, 1, 2])
def test_bits_are_those_of_separate_kernels(arch, seq, hd):
    import paper_2401_15207_amd as H
    wl = dict(WORKLOADS["C1"], arch=arch, n_classes=2 if arch == 1 else 0, batch=2, d_model=3 * hd, n_heads=3, d_ffn=40, max_seq=256)
    (la, a), (lb, b) = (_grads(wl, u, seq) for u in (0, H.UNFUSED_ATTENTION))
    assert np.array_equal(la, lb) and np.array_equal(a, b)


@pytest.mark.parametrize("seq", [8, 31])
@pytest.mark.parametrize("arch", [0, 1])
def test_gelu_on_the_way_out_changes_no_bit(arch, seq):
    import paper_2401_15207_amd as H
    wl = dict(WORKLOADS["C1"], arch=arch, n_classes=2 if arch == 1 else 0, batch=3, d_model=60, n_heads=3, d_ffn=131)
    (la, a), (lb, b) = (_grads(wl, u, seq) for u in (0, H.UNFUSED_EPILOGUES))
    assert np.array_equal(la, lb) and np.array_equal(a, b)


@pytest.mark.parametrize("batch,seq", [(1, 1), (1, 63), (1, 64), (1, 65), (3, 256), (7, 110), (4, 256), (5, 205), (4, 257), (7, 256), (16, 256), (17, 241)])
def test_column_sums_of_any_number_of_rows(batch, seq):
    """Gains and biases: one launch up to 1024 rows (two sums at once: 768), two beyond; chunks of 64 rows, whole and not, 12 and 16 of
    them and one more, several more, 64 and one more."""
    wl = dict(arch=1, n_layers=1, d_model=68, n_heads=1, d_ffn=20, vocab=64, max_seq=max(seq, 8), n_classes=2, norm_eps=1e-5, rope_base=10000.0,
              dtype=0, batch=batch, seq=seq, m=1, strategy="top2down", opt=SGD1)
    _compare_gradients(wl, 47)


@pytest.mark.parametrize("seq,hd,one_kernel", [(64, 16, True), (65, 16, False), (64, 64, True), (128, 64, False), (256, 32, False), (64, 68, False)])
def test_one_kernel_up_to_64_tokens(seq, hd, one_kernel):
    """Longer sequences take the separate contractions and softmax kernels, which are faster there."""
    import paper_2401_15207_amd as H
    wl = dict(WORKLOADS["C1"], batch=2, d_model=2 * hd, n_heads=2, d_ffn=40, max_seq=256)
    gpu = H.HiftModel(model_config(wl), SGD1, 1, 2, seq)
    gpu.set_group_schedule("bottom2up", 1)
    gpu.profile_enable(True)
    gpu.step(*to_dev(*make_batch(dict(wl, seq=seq), 43, 1)), 0)
    rows = gpu.profile_read_rowwise()
    launches = [n for name, (n, _ms, _bytes) in rows.items() if "softmax" in name]
    assert len(launches) == 2 and all((n == 0) == one_kernel for n in launches), rows
