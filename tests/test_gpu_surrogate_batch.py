"""Training windows run together against the same windows one after another, to the bit: the loss, the
last window's stored activations and the weight gradient (every sum keeps its order).  Also a batch
larger than the windows that fit together, and a workspace that grows."""
import numpy as np
import pytest
import torch

from paper_2507_21748_amd.surrogate import Net

pytestmark = pytest.mark.gpu


def _windows(b, n, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    x = torch.randn((b, n, n, n), generator=g, device="cuda").mul_(0.5)
    return x, (x + 0.1 * torch.randn((b, n, n, n), generator=g, device="cuda")).contiguous()


def _step(x, y, together):
    net = Net(seed=3)
    net.TRAIN_WINDOWS = together
    loss = float(net.train_step(x, y, 2, 1e-4).item())
    buf = {k: v.clone() for k, v in net.train_buffers(x.shape[1]).items()}
    return loss, buf


@pytest.mark.parametrize("b,n,together", [(2, 9, 8), (3, 16, 8), (4, 24, 3), (5, 21, 2)])
def test_windows_together_match_one_by_one(evx_gpu, b, n, together):
    print(f"windows together {b} x {n}^3, {together} at once", flush=True)
    x, y = _windows(b, n, 17)
    la, ba = _step(x, y, together)
    lb, bb = _step(x, y, 1)
    assert la == lb
    for k in ba:
        assert torch.equal(ba[k], bb[k]), k


def test_workspace_grows_with_the_batch(evx_gpu):
    net, ref = Net(seed=5), Net(seed=5)
    for b in (1, 3, 2, 4):
        x, y = _windows(b, 12, b)
        a = float(net.train_step(x, y, 2, 1e-4).item())
        ref._ws.clear()
        torch.cuda.synchronize()
        assert a == float(ref.train_step(x, y, 2, 1e-4).item())
    assert np.isfinite(a)
