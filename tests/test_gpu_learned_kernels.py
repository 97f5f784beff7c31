"""GPU: the network's kernels at the edges of their tiles, and rows that
share memory.

The training kernel takes tiles of 16 samples, at most 128 work-groups at a
time: one sample, one tile and its neighbours, the last size with one tile
per work-group and the first with more, and a size with several tiles each.
Tolerances are those of the larger gradient test: FP32 sums of n terms
against FP64, 1e-5 of the loss and 1e-4 of the largest gradient entry.
"""

import ctypes as C

import numpy as np
import pytest

from oracle import learned as L
from paper_2606_15720_amd import ugks as U
from paper_2606_15720_amd import warmstart as WS
from test_zz_no_alloc import D2H, H2D, _hip

pytestmark = pytest.mark.gpu


def _net(seed):
    rng = np.random.default_rng(seed)
    p = (WS.init_params(seed) + rng.normal(0, 0.05, WS.NPARAM)).astype(np.float32)
    si = rng.uniform(0.5, 2.0, 9).astype(np.float32)
    so = rng.uniform(0.5, 2.0, 9).astype(np.float32)
    return p, si, so


@pytest.mark.parametrize("n", [1, 15, 16, 17, 2048, 2049, 5000])
def test_loss_and_gradient_at_tile_edges(n):
    p, si, so = _net(8)
    rng = np.random.default_rng(n)
    x = rng.normal(0.0, 1.0, (n, 9)).astype(np.float32)
    t = rng.normal(0.0, 1.0, (n, 9)).astype(np.float32)
    net = U.MLP(p, si, so)
    loss, grad = net.loss_grad(x, t)
    lo, go = L.loss_grad(p.astype(np.float64), (x * si).astype(np.float64), (t / so).astype(np.float64))
    rel = np.abs(grad - go).max() / np.abs(go).max()
    print(n, "loss", loss, lo, "grad", rel, flush=True)
    assert loss == pytest.approx(lo, rel=1e-5)
    assert rel <= 1e-4
    again = net.loss_grad(x, t)
    assert again[0] == loss and np.array_equal(again[1], grad)
    net.close()


@pytest.mark.parametrize("entry", ["forward_device", "forward_noalloc"])
@pytest.mark.parametrize("shift", [0, 9, -13])
def test_inference_on_rows_that_share_memory(entry, shift):
    # outputs in place of the inputs, and outputs that overlap them
    hip = _hip()
    assert hip.hipSetDevice(0) == 0
    p, si, so = _net(9)
    rows, pad = 1037, 64
    x = np.random.default_rng(1).normal(0.0, 0.7, (rows, 9)).astype(np.float32)
    net = U.MLP(p, si, so)
    ref = net.forward(x)
    host = np.zeros(rows * 9 + 2 * pad, dtype=np.float32)
    host[pad:pad + rows * 9] = x.ravel()
    buf = C.c_void_p()
    assert hip.hipMalloc(C.byref(buf), host.nbytes) == 0
    assert hip.hipMemcpy(buf, host.ctypes.data_as(C.c_void_p), host.nbytes, H2D) == 0
    at = buf.value + 4 * pad
    getattr(net, entry)(at, rows, at + 4 * shift)
    assert hip.hipDeviceSynchronize() == 0
    assert hip.hipMemcpy(host.ctypes.data_as(C.c_void_p), buf, host.nbytes, D2H) == 0
    assert np.array_equal(host[pad + shift:pad + shift + rows * 9].reshape(rows, 9), ref)
    hip.hipFree(buf)
    net.close()
