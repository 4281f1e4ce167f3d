"""The trainer's gradient kernel at the edges of its row split (rows per wave,
rows per block, blocks per batch) against the NumPy FP64 oracle, and an epoch
against the same batches taken one by one.

Bars: gradient within 1e-4 of its largest entry and loss within 1e-5, as for
the whole-batch test: an FP32 sum of B terms in any order is off by at most
B 2^-24 of its terms' magnitudes, 2.5e-4 of them at B = 4,100 and far less in
the blocked order, and the terms' magnitudes are of the largest entry's size.
"""
import numpy as np
import pytest

from oracle import mlp as omlp
from test_gpu_mlp import _data

pytestmark = [pytest.mark.gpu, pytest.mark.filterwarnings("ignore::RuntimeWarning")]


@pytest.mark.parametrize("B,max_batch", [(1, 1), (3, 7), (4, 4), (5, 1025), (8, 8), (9, 16), (1023, 1023), (1025, 1025), (2048, 2048),
                                         (2049, 4100), (4100, 4100)])
def test_gradient_row_split(B, max_batch):
    from paper_2608_22269_amd import learn
    X, y, w, mean, std, th = _data(11 + B, B)
    tr = learn.MLPTrainer(th, mean, std, max_batch=max_batch)
    for weights in (w, None):
        loss, g = tr.loss_grad(X, y, weights)
        rl, rg = omlp.loss_and_grad(th.astype(np.float64), X, y, np.ones(B) if weights is None else w, mean, std)
        assert abs(loss - rl) <= 1e-5 * abs(rl)
        assert np.abs(g - rg).max() <= 1e-4 * np.abs(rg).max()
    assert np.array_equal(tr.loss_grad(X, y, w)[1], tr.loss_grad(X, y, w)[1])


def test_epoch_equals_its_batches():
    """train_epoch (rows by permutation, update fused with the sum of the
    blocks) against loss_grad and adam of the same rows in the same order, the
    last batch ragged; FP32 rounding of the update: 2^-23 of a parameter a
    step."""
    import torch
    from paper_2608_22269_amd import learn
    n, batch = 2500, 1024
    X, y, w, mean, std, th = _data(5, n)
    perm = np.random.default_rng(6).permutation(n).astype(np.int32)
    a = learn.MLPTrainer(th, mean, std, max_batch=batch)
    b = learn.MLPTrainer(th, mean, std, max_batch=batch)
    up = lambda v: torch.as_tensor(v, device="cuda")  # noqa: E731
    mean_loss = a.train_epoch(up(X), up(y), up(w), up(perm), batch, 2e-3)
    losses = []
    for o in range(0, n, batch):
        r = perm[o:o + batch]
        losses.append(b.loss_grad(X[r], y[r], w[r])[0])
        b.adam(lr=2e-3)
    assert abs(mean_loss - np.mean(losses)) <= 1e-6 * abs(mean_loss)
    pa, pb = a.params(), b.params()
    assert np.abs(pa - pb).max() <= 3 * 2.0 ** -23 * np.abs(pb).max()
