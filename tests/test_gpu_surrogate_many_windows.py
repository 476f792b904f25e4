"""A training workspace of more windows than run together, through the C ABI: the windows past that
many stay untouched, and the batch's results are those of a one-window workspace to the bit."""
import ctypes

import pytest
import torch

from paper_2507_21748_amd import evx
from paper_2507_21748_amd.surrogate import Net

pytestmark = pytest.mark.gpu

EDGE, BATCH, TOGETHER = 3, 1026, 1024


def _bytes(windows):
    nb = ctypes.c_size_t()
    evx._check(evx._LIB.evx_surrogate_workspace_bytes(EDGE, EDGE, EDGE, windows, ctypes.byref(nb)),
               "evx_surrogate_workspace_bytes")
    return nb.value


def _train(x, y, nbytes):
    net = Net(seed=3)
    ws = torch.full((nbytes + 256,), 0x5A, dtype=torch.uint8, device="cuda")
    off = -ws.data_ptr() % 256
    evx._check(evx._LIB.evx_surrogate_train_step(
        net._h, evx._dev_ptr(x), evx._dev_ptr(y), BATCH, EDGE, 1, evx._dev_ptr(net.params),
        evx._dev_ptr(net.m), evx._dev_ptr(net.v), 1, 1e-4, evx._dev_ptr(net.loss, torch.float64, 1),
        ctypes.c_void_p(ws.data_ptr() + off), nbytes, evx._stream_handle()),
        "evx_surrogate_train_step")
    return net, ws[off:off + nbytes]


def test_windows_past_the_limit(evx_gpu):
    print(f"{BATCH} windows of {EDGE}^3", flush=True)
    g = torch.Generator(device="cuda").manual_seed(5)
    x = torch.randn((BATCH, EDGE, EDGE, EDGE), generator=g, device="cuda").mul_(0.5)
    y = (x * 0.9).contiguous()
    one, _ = _train(x, y, _bytes(1))
    net, ws = _train(x, y, _bytes(BATCH))
    assert bool((ws[_bytes(TOGETHER):] == 0x5A).all())
    assert torch.equal(net.loss, one.loss)
    for a, b in ((net.params, one.params), (net.m, one.m), (net.v, one.v)):
        assert torch.equal(a, b)
