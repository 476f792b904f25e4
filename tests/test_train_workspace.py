"""The training workspace of the binding without a GPU (host memory stands for the device's): fewer
windows at once when the memory for all of them is not there, one window at least, and a workspace
that a larger one replaces stays until the workspaces are released, since a captured graph, another
stream or a view of its buffers may still use it."""
import ctypes
import gc
import weakref

import pytest
import torch

from paper_2507_21748_amd import evx, surrogate

N = 9  # window edge


@pytest.fixture
def net():
    surrogate._lib()
    net = surrogate.Net.__new__(surrogate.Net)
    net.device, net._ws = "cpu", {}
    return net


def size(windows):
    nb = ctypes.c_size_t()
    assert evx._LIB.evx_surrogate_workspace_bytes(N, N, N, windows, ctypes.byref(nb)) == 0
    return nb.value


def windows_of(ws):
    return 1 + (ws.nbytes - size(1)) // (size(2) - size(1))


@pytest.fixture
def limit(monkeypatch):
    """Allocations above limit.nbytes fail as a full device's do."""
    made = surrogate._Workspace

    def make(nbytes, *a):
        limit.calls += 1
        if nbytes > limit.nbytes:
            raise torch.OutOfMemoryError("out of memory")
        return made(nbytes, *a)

    limit.calls, limit.nbytes = 0, 1 << 60
    monkeypatch.setattr(surrogate, "_Workspace", make)
    return limit


@pytest.mark.parametrize("batch,room,expect", [(4, 4, 4), (8, 7, 4), (8, 3, 2), (6, 1, 1), (1, 1, 1)])
def test_fewer_windows_when_memory_is_short(net, limit, batch, room, expect):
    limit.nbytes = size(room)
    ws = net._workspace((N, N, N), batch)
    assert windows_of(ws) == expect
    calls = limit.calls
    assert net._workspace((N, N, N), batch) is ws and limit.calls == calls  # no try on every step


def test_no_window_fits(net, limit):
    limit.nbytes = size(1) - 1
    with pytest.raises(torch.OutOfMemoryError):
        net._workspace((N, N, N), 4)


def test_smaller_workspace_kept_when_a_larger_one_does_not_fit(net, limit):
    first = net._workspace((N, N, N), 2)
    limit.nbytes = size(2)
    assert net._workspace((N, N, N), 8) is first


def test_replaced_workspace_stays_until_released(net):
    first = weakref.ref(net._workspace((N, N, N), 1).buf)
    assert windows_of(net._workspace((N, N, N), 4)) == 4
    gc.collect()
    assert first() is not None
    net.release_workspaces()
    gc.collect()
    assert first() is None


def test_one_inference_workspace_per_shape(net):
    ws = net._workspace((N, N, N), 0)
    assert net._workspace((N, N, N), 0) is ws is not net._workspace((N, N, N), 2)
