"""Gradient of the token table where the lists of positions are at their edges: a row's positions spread over two batches of tokens, batches as long as the
lists of each length,
their number around the rows read together, widths with and without whole pieces of four, a last piece of columns partly empty.
Against the oracle; plain SGD at rate 1 writes the gradient into the weights."""
import numpy as np
import pytest

from oracle import hift_oracle as O
from tests.hift_pair import make_pair, rel_l2, to_dev

pytestmark = pytest.mark.gpu

SGD1 = dict(kind="sgd", lr=1.0, beta1=0, beta2=0, eps=0, weight_decay=0.0, momentum=0.0)


@pytest.mark.parametrize("d,heads,batch,seq,tied", [(6, 1, 29, 73, 0), (8, 2, 29, 73, 0), (8, 2, 29, 73, 1), (1032, 3, 2, 24, 0), (1032, 3, 2, 24, 1),
                                                    (1026, 3, 2, 24, 0),
                                                    (8, 2, 8, 32, 0), (6, 1, 1, 257, 0), (6, 1, 4, 256, 0), (8, 2, 5, 205, 0)])
def test_rows_of_repeated_tokens(d, heads, batch, seq, tied):
    wl = dict(arch=0, n_layers=1, d_model=d, n_heads=heads, d_ffn=16, vocab=23, max_seq=seq, n_classes=0, norm_eps=1e-5,
              rope_base=10000.0, dtype=0, tie_embeddings=tied, batch=batch, seq=seq, m=1, strategy="bottom2up", opt=SGD1)
    # token v occurs v times (0, 1, ... 20: on both sides of 4, 8 and 16 rows at a time), token 21 at the very end, 22 everywhere else
    rng = np.random.default_rng(3)
    n = batch * seq
    tok = np.full(n, 22, np.int32)
    at = rng.permutation(n - 1)
    i = 0
    for v in range(min(21, int((2 * (n - 8)) ** 0.5))):
        tok[at[i:i + v]] = v
        i += v
    tok[-1] = 21
    tok = tok.reshape(batch, seq)
    lab = np.full_like(tok, -1)
    lab[:, :-1] = tok[:, 1:]
    orc, gpu, theta0 = make_pair(wl, seed=11, opt=SGD1, jitter=0.02)
    _loss, g = O.loss_and_grad(orc.cfg, theta0.astype(np.float64), tok, lab)
    gpu.step(*to_dev(tok, lab), 0)
    lo, hi = orc.group_range(0)
    got = (theta0.astype(np.float64) - gpu.read_params().astype(np.float64))[lo:hi]
    rows, ref = got[:23 * d].reshape(23, d), g[lo:hi][:23 * d].reshape(23, d)
    # the difference of two weights near 1 in fp32 holds a gradient to 6e-8 of the weights (jitter: up to 0.1)
    slack = 1.2e-7 * np.abs(theta0[lo:hi][:23 * d]).max()
    for v in range(23):
        assert np.linalg.norm(rows[v] - ref[v]) <= 3e-5 * np.linalg.norm(ref[v]) + slack * d ** 0.5 * 3, v
    assert rel_l2(rows, ref) <= 3e-5
