"""Calls of the network that a faster path must not make slower or refuse."""
import time

import numpy as np
import pytest

from tests.test_gpu_mlp import M, _data, _norm, _params  # noqa: F401  (M: fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [8192, 8193, 20000])
def test_host_rows_by_either_way(M, rows):  # noqa: F811
    import torch
    X, _ = _data(rows, seed=rows)
    nrm, _ = _norm(M, *_data(100))
    net = M.Mlp(_params(5), nrm, max_batch=rows)
    assert np.array_equal(net.forward(X), net.forward(torch.as_tensor(X, device="cuda")))
    with pytest.raises(ValueError):
        net.forward(X[:, :2])
    with pytest.raises(M.LbmError):
        net.forward(np.concatenate([X, X]))       # more rows than max_batch
    net.close()


def test_many_host_rows_cost_what_a_copy_and_a_launch_do(M):  # noqa: F811
    import torch
    X, _ = _data(300_000, seed=1)
    nrm, _ = _norm(M, *_data(100))
    net = M.Mlp(_params(5), nrm, max_batch=len(X))

    def shortest(f):
        best = float("inf")
        for _ in range(12):
            t0 = time.perf_counter()
            f()
            best = min(best, time.perf_counter() - t0)
        return best

    copy = shortest(lambda: net.forward(torch.as_tensor(X, device="cuda")))
    host = shortest(lambda: net.forward(X))
    net.close()
    assert host < 1.5 * copy, (host, copy)        # in pieces of 4,096 rows: 3 times


@pytest.mark.parametrize("every", [-5, 5.0, -1])
def test_train_logs_at_any_multiple(M, every):  # noqa: F811
    # a step s is logged where s % log_every is 0, and the last one
    X, T = _data(200, seed=4)
    nrm, _ = _norm(M, X, T)
    a, b = (M.Mlp(_params(2), nrm, max_batch=32) for _ in range(2))
    want = a.train(X, T, steps=13, lr=1e-3, batch=32, log_every=abs(int(every)))
    got = b.train(X, T, steps=13, lr=1e-3, batch=32, log_every=every)
    assert got == want and [s for s, _ in want] == [s for s in range(13) if s % every == 0 or s == 12]
    assert np.array_equal(a.params(), b.params())
    a.close(); b.close()
