"""The network's multi-step and host entry points: gathered minibatch steps equal one
gradient and one Adam step at a time on the gathered rows, bit for bit, and the host
forward pass equals the device one, at sizes around the 32-row tiles, the 256
gradient work-groups and the 4096-row staging buffer."""
import ctypes as C

import numpy as np
import pytest

from tests.test_gpu_mlp import M, _data, _norm, _params  # noqa: F401  (M: fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch", [1, 32, 33, 777, 8225])
def test_gathered_steps_equal_single_steps(M, batch):  # noqa: F811
    import torch
    n, steps = max(64, 2 * batch), 4
    X, T = _data(n, seed=batch)
    nrm, _ = _norm(M, X, T)
    a = M.Mlp(_params(2), nrm, max_batch=batch)
    b = M.Mlp(_params(2), nrm, max_batch=batch)
    idx = np.random.default_rng(3).integers(0, n, size=(steps, batch))
    lrs = [2e-3, 1e-3, 5e-4, 1e-4]
    losses = []
    for i in range(steps):
        loss, g = a.gradient(X[idx[i]], T[idx[i]])
        losses.append(loss)
        a.adam(g, lrs[i])
    Xd, Td = torch.as_tensor(X, device="cuda"), torch.as_tensor(T, device="cuda")
    di = torch.as_tensor(idx, device="cuda")
    torch.cuda.synchronize()
    lr = (C.c_float * steps)(*lrs)
    assert M.lib().mlp_train_steps(b.ctx, Xd.data_ptr(), Td.data_ptr(), di.data_ptr(), batch, steps,
                                   C.addressof(lr), b.loss.data_ptr()) == 0
    assert np.array_equal(a.params(), b.params())
    assert float(b.loss.cpu()[0]) == losses[-1]
    # refused: no steps, too many rows, a rate that is not positive
    bad = (C.c_float * 2)(1e-3, 0.0)
    for args in [(batch, 0, lr), (batch + 1, 1, lr), (batch, 2, bad)]:
        assert M.lib().mlp_train_steps(b.ctx, Xd.data_ptr(), Td.data_ptr(), di.data_ptr(), args[0], args[1],
                                       C.addressof(args[2]), None) != 0
    assert np.array_equal(a.params(), b.params())
    a.close(); b.close()


@pytest.mark.parametrize("B", [1, 32, 4001, 4096, 4097, 9000])
def test_host_forward_equals_device_forward(M, B):  # noqa: F811
    import torch
    X, T = _data(B, seed=B)
    nrm, _ = _norm(M, *_data(100))
    net = M.Mlp(_params(5), nrm, max_batch=B)
    y = net.forward(X)
    assert np.array_equal(y, net.forward(torch.as_tensor(X, device="cuda")))
    assert np.array_equal(y, net.forward(X))
    net.close()


def test_host_forward_from_two_threads(M):  # noqa: F811
    from concurrent.futures import ThreadPoolExecutor
    xs = [_data(4096, seed=s)[0] for s in (1, 2)]
    nrm, _ = _norm(M, *_data(100))
    net = M.Mlp(_params(5), nrm, max_batch=4096)
    want = [net.forward(x) for x in xs]
    with ThreadPoolExecutor(2) as pool:
        for i, y in enumerate(pool.map(lambda i: net.forward(xs[i % 2]), range(200))):
            assert np.array_equal(y, want[i % 2]), i
    net.close()


def test_train_refuses_fewer_targets_than_rows(M):  # noqa: F811
    X, T = _data(64, seed=1)
    nrm, _ = _norm(M, X, T)
    net = M.Mlp(_params(2), nrm, max_batch=32)
    with pytest.raises(IndexError):
        net.train(X, T[:40], steps=2, lr=1e-3, batch=32)
    net.close()
