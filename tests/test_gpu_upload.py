"""The classifier's weights in one transfer (32- and 64-bit floats) or one
each (other kinds): the same logits bit for bit, and an empty array is refused
as before."""
import numpy as np
import pytest

from test_gpu_mlp import _data

pytestmark = [pytest.mark.gpu, pytest.mark.filterwarnings("ignore::RuntimeWarning")]


@pytest.mark.parametrize("name", ["infer_bf16", "forward_noalloc"])
def test_kinds_of_weights(name):
    from paper_2608_22269_amd import _lib as L, learn
    import torch
    fn = getattr(learn, name)
    X, _, _, mean, std, th = _data(4, B=65)
    th, mean, std = th.astype(np.float16), mean.astype(np.float16), std.astype(np.float16)
    X = torch.as_tensor(X, device="cuda")
    ref = fn(th, mean, std, X).cpu().numpy()  # one transfer each
    for dt in (np.float32, np.float64):
        got = fn(th.astype(dt), mean.astype(np.float32),
                 list(std.astype(np.float64)), X).cpu().numpy()
        assert np.array_equal(got, ref), dt
    strided = np.zeros((2, len(th)), np.float32)
    strided[1] = th
    assert np.array_equal(fn(strided[1], np.repeat(mean.astype(np.float32), 2)[::2], std.astype(np.float64),
                             X).cpu().numpy(), ref)
    with pytest.raises(L.SphError):
        fn(th.astype(np.float32), np.zeros(0, np.float32), std.astype(np.float32), X)
