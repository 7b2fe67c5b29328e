"""A training step's loss arrives the same in a pinned word (written by the
device), in a pageable one (copied) and in another thread; without one the
call does not wait.  The gradient is the same bits each time."""
import ctypes
import threading

import numpy as np
import pytest

import oracle
from gpu_common import dn, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 257])
def test_every_way_to_the_loss(n):
    import torch
    D = dn()
    rng = np.random.default_rng(n)
    tiles = rng.normal(0, 0.5, (n, 2, 10, 10, 10)).astype(np.float32)
    targets = rng.normal(0, 0.5, (n, 512)).astype(np.float32)
    mask = (rng.random((n, 512)) < 0.5).astype(np.float32)
    prm = rng.normal(0, 0.12, D.NET_PARAMS).astype(np.float32)
    args = [to_dev(a, torch.float32) for a in (tiles, prm, targets, mask)]
    grads = [torch.full((D.NET_PARAMS,), float("nan"), device="cuda") for _ in range(4)]
    a = D.net_loss_grad(*args, grads[0], kind=0)
    other = []
    t = threading.Thread(target=lambda: other.append(D.net_loss_grad(*args, grads[1], kind=0)))
    t.start()
    t.join()
    word = ctypes.c_double(-1)
    ws, nbytes = D.workspace("net_train", D.lib().dn_net_bytes(n, 1))
    D.check(D.lib().dn_net_loss_grad(*(D._ptr(args[k]) for k in (0,)), n, *(D._ptr(args[k]) for k in (1, 2, 3)), 0,
                                     D._ptr(grads[2]), ws, nbytes, ctypes.byref(word),
                                     ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)))
    assert D.net_loss_grad(*args, grads[3], kind=0, sync=False) is None
    torch.cuda.synchronize()
    assert a == other[0] == word.value
    assert all(torch.equal(grads[0], g) for g in grads[1:])
    ref, _ = oracle.net_loss_grad(tiles.astype(np.float64), prm.astype(np.float64), targets.astype(np.float64),
                                  mask.astype(np.float64), kind=0, gate=1)
    assert abs(a - ref) <= 5e-3 * abs(ref)
