"""Front end of the learned free-surface classifier entry points of the C ABI
(training object, BF16 inference) and of the data it learns from.  All
arithmetic runs in libwbsph.so; this module marshals torch device buffers."""
from __future__ import annotations

import ctypes as C

import numpy as np

from . import _lib as L
from .sim import Simulation, _check, device_buffer

NFEAT = 16
NPARAM = L.MLP_NPARAM


def _dev(a, dtype=None):
    import torch
    t = torch.as_tensor(np.ascontiguousarray(a), device="cuda")
    return t if dtype is None else t.to(dtype)


def _upload(*arrays):
    """Float32 copies of small arrays on the device: the tensors that hold them
    and their addresses.  Arrays of 32- and 64-bit floats go in one transfer
    (each waits for the device, some 14 us: 66 us for a forward pass of 1,000
    rows with three, 36 us with one), each at a multiple of 256 bytes."""
    import torch
    host = [np.ascontiguousarray(a) for a in arrays]
    if any(a.dtype not in (np.float32, np.float64) or a.size == 0 for a in host):
        dev = [_dev(a, torch.float32) for a in host]
        return dev, [t.data_ptr() for t in dev]
    at = np.cumsum([0] + [-(-a.size // 64) * 64 for a in host])
    buf = np.empty(at[-1], np.float32)
    with np.errstate(all="ignore"):  # beyond float32's range: infinite, as torch converts
        for a, o in zip(host, at):
            buf[o:o + a.size] = a.ravel()
    t = torch.as_tensor(buf, device="cuda")
    return [t], [t.data_ptr() + 4 * int(o) for o in at[:-1]]


def _lend(stream, *tensors):
    """Before a launch on `stream`, if that is not the current one: it starts
    after what the current stream has been given, and the memory of the
    tensors (None: skipped), which belongs to the current stream, is not given
    away there while `stream` still works on it."""
    import torch
    cur = torch.cuda.current_stream()
    if stream == cur:
        return
    stream.wait_stream(cur)
    for t in tensors:
        if t is not None:
            t.record_stream(stream)


def _returned(stream):
    """After a launch on `stream`: the current stream waits for it."""
    import torch
    cur = torch.cuda.current_stream()
    if stream != cur:
        cur.wait_stream(stream)


class MLPTrainer:
    """FP32 trainer (hand-written HIP forward, backward and Adam kernels)."""

    def __init__(self, params0, mean, std, max_batch=4096, stream=None):
        import torch
        self.torch = torch
        lib = L.lib()
        nbytes = lib.sph_mlp_workspace_bytes(int(max_batch))
        if nbytes == 0:
            raise L.SphError(L.SPH_EINVAL, "sph_mlp_workspace_bytes")
        self._ws, ptr = device_buffer(nbytes)
        cur = torch.cuda.current_stream()
        self.stream = stream if stream is not None else cur
        self._side = self.stream != cur
        _lend(self.stream, self._ws)
        p0 = np.ascontiguousarray(params0, dtype=np.float32)
        mu = np.ascontiguousarray(mean, dtype=np.float32)
        sd = np.ascontiguousarray(std, dtype=np.float32)
        self.mean, self.std = mu, sd
        h = C.c_void_p()
        pp = lambda a: a.ctypes.data_as(C.c_void_p)
        _check(lib.sph_mlp_create(int(max_batch), pp(p0), pp(mu), pp(sd), C.c_void_p(ptr), nbytes,
                                  C.c_void_p(self.stream.cuda_stream), C.byref(h)), "sph_mlp_create")
        self.h = h
        self.max_batch = int(max_batch)

    def close(self):
        if getattr(self, "h", None):
            L.lib().sph_mlp_destroy(self.h)
            self.h = None

    def __del__(self):
        try:
            self.close()
        except Exception:
            pass

    def forward(self, X):
        X = _dev(X, self.torch.float32)
        out = self.torch.empty(X.shape[0], dtype=self.torch.float32, device="cuda")
        _lend(self.stream, X, out)
        _check(L.lib().sph_mlp_forward(self.h, C.c_void_p(X.data_ptr()), X.shape[0], C.c_void_p(out.data_ptr())),
               "sph_mlp_forward")
        _returned(self.stream)
        return out.cpu().numpy()

    def loss_grad(self, X, y, w=None):
        torch = self.torch
        X = _dev(X, torch.float32)
        y = _dev(y, torch.float32)
        wd = None if w is None else _dev(w, torch.float32)
        loss = torch.empty(1, dtype=torch.float32, device="cuda")
        grad = torch.empty(NPARAM, dtype=torch.float32, device="cuda")
        _lend(self.stream, X, y, wd, loss, grad)
        _check(L.lib().sph_mlp_loss_grad(self.h, C.c_void_p(X.data_ptr()), C.c_void_p(y.data_ptr()),
                                         C.c_void_p(wd.data_ptr()) if wd is not None else None, X.shape[0],
                                         C.c_void_p(loss.data_ptr()), C.c_void_p(grad.data_ptr())),
               "sph_mlp_loss_grad")
        _returned(self.stream)
        return float(loss.item()), grad.cpu().numpy()

    def adam(self, lr=1e-3, beta1=0.9, beta2=0.999, eps=1e-8):
        _check(L.lib().sph_mlp_adam(self.h, lr, beta1, beta2, eps), "sph_mlp_adam")

    def train_epoch(self, Xd, yd, wd, perm_d, batch, lr):
        """One epoch over device tensors (X n x 16 f32, y, w f32, perm int32)."""
        ml = C.c_float(0.0)
        if self._side:  # asking for the current stream takes 3 us of some 320
            _lend(self.stream, Xd, yd, wd, perm_d)
        _check(L.lib().sph_mlp_train_epoch(self.h, C.c_void_p(Xd.data_ptr()), C.c_void_p(yd.data_ptr()),
                                           C.c_void_p(wd.data_ptr()) if wd is not None else None,
                                           C.c_void_p(perm_d.data_ptr()), Xd.shape[0], int(batch), float(lr),
                                           C.byref(ml)), "sph_mlp_train_epoch")
        return ml.value

    def params(self):
        out = np.empty(NPARAM, dtype=np.float32)
        _check(L.lib().sph_mlp_get_params(self.h, out.ctypes.data_as(C.c_void_p), 0), "sph_mlp_get_params")
        return out


def infer_bf16(params, mean, std, X, stream=None):
    """Logits of the rows of X with BF16 MFMA inference (device tensors or
    arrays), on `stream` (the current one) and ready in its order."""
    return _logits(L.lib().sph_mlp_infer_bf16, "sph_mlp_infer_bf16", params, mean, std, X, stream)


def forward_noalloc(params, mean, std, X, stream=None):
    """FP32 logits of the rows of X through sph_mlp_forward_noalloc (the
    trainer's forward pass without a trainer or workspace; at most
    SPH_MLP_NOALLOC_MAX_ROWS rows), on `stream` (the current one) and ready in
    its order.  Returns a device tensor."""
    return _logits(L.lib().sph_mlp_forward_noalloc, "sph_mlp_forward_noalloc", params, mean, std, X, stream)


def _logits(call, what, params, mean, std, X, stream):
    import torch
    hold, (w, mu, sd) = _upload(params, mean, std)
    Xd = X if isinstance(X, torch.Tensor) else _dev(X, torch.float32)
    out = torch.empty(Xd.shape[0], dtype=torch.float32, device="cuda")
    if stream is None:
        s = torch.cuda.current_stream()
    else:
        s = stream
        _lend(s, *hold, Xd, out)
    _check(call(C.c_void_p(w), C.c_void_p(mu), C.c_void_p(sd), C.c_void_p(Xd.data_ptr()), Xd.shape[0],
                C.c_void_p(out.data_ptr()), C.c_void_p(s.cuda_stream)), what)
    return out


def candidate_samples(sim: Simulation):
    """Features and exact labels of the particles the scan-region pass decided
    in the last right-hand side (lambda between the two thresholds)."""
    path = sim.field("fs_path")
    sel = path == 1
    feats = sim.field("features")[sel]
    labels = sim.field("fs")[sel].astype(np.float32)
    return feats, labels
