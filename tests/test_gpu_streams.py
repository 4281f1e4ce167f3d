"""Classifier calls on a stream of the caller's that still has work to do:
what they upload and return lies in memory of the current stream, which must
not pass to the next call before they have run.  Bit for bit against the same
calls on the current stream."""
import numpy as np
import pytest

from test_gpu_mlp import _data

pytestmark = [pytest.mark.gpu, pytest.mark.filterwarnings("ignore::RuntimeWarning")]


def _busy(stream, a):
    """Some milliseconds of work on the stream."""
    import torch
    stream.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(stream):
        for _ in range(20):
            a = a @ a
    return a


@pytest.fixture(scope="module")
def load():
    import torch
    return torch.eye(4096, device="cuda")


@pytest.mark.parametrize("name", ["infer_bf16", "forward_noalloc"])
def test_calls_in_a_row_on_a_side_stream(name, load):
    import torch
    from paper_2608_22269_amd import learn
    fn = getattr(learn, name)
    sets = [_data(seed, B=777) for seed in range(4)]
    ref = [fn(th, mean, std, X).cpu().numpy() for X, _, _, mean, std, th in sets]
    side = torch.cuda.Stream()
    held = _busy(side, load)
    got = [fn(th, mean, std, X, stream=side) for X, _, _, mean, std, th in sets]
    scrap = [torch.full((777,), np.nan, device="cuda") for _ in range(8)]  # on the current stream
    side.synchronize()
    for g, r in zip(got, ref):
        assert np.array_equal(g.cpu().numpy(), r)
    del held, scrap


def test_trainer_on_a_side_stream(load):
    import torch
    from paper_2608_22269_amd import learn
    X, y, w, mean, std, th = _data(9, B=600)
    a = learn.MLPTrainer(th, mean, std, max_batch=600)
    ref, (loss, grad) = a.forward(X), a.loss_grad(X, y, w)
    side = torch.cuda.Stream()
    b = learn.MLPTrainer(th, mean, std, max_batch=600, stream=side)
    held = _busy(side, load)
    assert np.array_equal(b.forward(X), ref)
    held = _busy(side, load)
    loss_b, grad_b = b.loss_grad(X, y, w)
    assert loss_b == loss and np.array_equal(grad_b, grad)
    ptr = b._ws.data_ptr()
    held = _busy(side, load)
    nbytes = b._ws.numel()
    b.close()
    del b  # its workspace is free once the side stream has passed this point
    other = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    busy = not side.query()
    assert not busy or other.data_ptr() != ptr
    side.synchronize()
    del held, other


def test_simulation_on_a_side_stream(load):
    """Steps queued behind other work on a side stream, the context dropped
    before they have run: its workspace is not handed out meanwhile, and the
    field they export last is that of the current stream's steps."""
    import torch
    import workloads as wl
    from paper_2608_22269_amd import Simulation
    case = wl.random_velocity(wl.tank2d(dx=0.02), 0.05, 3)
    a = Simulation(case)
    a.step(3)
    ref = a.field("x")
    side = torch.cuda.Stream()
    b = Simulation(case, stream=side)
    out = torch.zeros(ref.shape, dtype=torch.float64, device="cuda")
    held = _busy(side, load)
    b.step(3)
    b.field_device("x", out)
    ptr, nbytes = b._ws.data_ptr(), b._ws.numel()
    b.close()
    del b
    other = torch.empty(nbytes, dtype=torch.uint8, device="cuda").fill_(255)
    busy = not side.query()
    assert not busy or other.data_ptr() != ptr
    side.synchronize()
    assert np.array_equal(out.cpu().numpy(), ref)
    a.close()
    del held, other
