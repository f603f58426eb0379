"""Inference at the ends of its tiles of rows and of its pieces of 2^20 rows, from a workspace that
calls of several sizes and threads share: a row's outputs do not depend on the rows around it."""
import threading

import numpy as np
import pytest

from paper_1608_01125_amd import tril as T

from test_gpu_mlp import torch  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("members", [1, 3])
@pytest.mark.parametrize("n", [1, 15, 79, 80, 81, 160, 241, (1 << 20) + 81])
def test_rows_do_not_depend_on_their_tile(torch, n, members):  # noqa: F811
    rng = np.random.default_rng(n)
    x = torch.from_numpy(rng.normal(0, 1, (n, 6)).astype(np.float32)).cuda()
    net = T.Mlp(members, seed=2)
    try:
        mean, sdev = net.predict(x)
        at = sorted({0, n // 2, n - 1} | ({1 << 20, (1 << 20) - 1} if n > 1 << 20 else set()))
        for i in at:  # a call of its own, in row 0 of its tile
            m1, s1 = net.predict(x[i:i + 1].contiguous())
            assert torch.equal(m1[0], mean[i]) and torch.equal(s1[0], sdev[i])
        if members == 1:
            assert not sdev.any()
    finally:
        net.close()


def test_threads_share_a_model(torch):  # noqa: F811
    rng = np.random.default_rng(9)
    xs = [torch.from_numpy(rng.normal(0, 1, (n, 6)).astype(np.float32)).cuda()
          for n in (70000, 333, 20000, 81)]
    net = T.Mlp(4, seed=3)
    try:
        want = [net.predict(x) for x in xs]
        torch.cuda.synchronize()
        got = [[] for _ in xs]

        def work(i):
            for _ in range(10):
                got[i].append(net.predict(xs[i]))

        threads = [threading.Thread(target=work, args=(i,)) for i in range(len(xs))]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        for w, g in zip(want, got):
            assert len(g) == 10
            assert all(torch.equal(w[0], a) and torch.equal(w[1], b) for a, b in g)
    finally:
        net.close()
