"""Voxels far apart in a map of just their number: more empty neighbours than the
map keeps rows for, so that searches probe instead, with the same answers as in a
roomy map, and an insert that stays linear."""
import time

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def lattice(n, side=40):
    """n points 4 m apart."""
    i = np.arange(n)
    x = np.stack([i % side, i // side % side, i // side ** 2]).astype(np.float32)
    return torch.from_numpy(4.0 * x + 0.5).cuda()


@pytest.mark.parametrize("n", [1, 30, 400, 4000, 30000])
def test_isolated_voxels(n):
    from paper_2606_26010_amd import far
    g = np.random.default_rng(n)
    x = lattice(n)
    q = x[:, torch.from_numpy(g.integers(0, n, 5000)).cuda()].contiguous()
    q += torch.from_numpy(g.uniform(-1.4, 1.4, (3, 5000)).astype(np.float32)).cuda()
    got = []
    for cap in (n, 16 * n):
        m = far.Map(1.0, 20, -1.0, cap, cap, 1)
        half = x[:, :n // 2].contiguous()
        torch.cuda.synchronize()
        t = time.perf_counter()
        assert n == 1 or m.insert(half)[1] == n // 2
        assert m.insert(x)[1] == n - n // 2
        ms = 1e3 * (time.perf_counter() - t)
        print(f"{n} voxels, capacity {cap}: {ms:.2f} ms")
        assert ms < 100.0
        cov, val = far.far_scan_covariances(q, 1.0, 5)
        lin = m.linearize(q, cov, val, np.eye(4), 1.0, 0.5, want_corr=True)
        got.append([*m.knn(q, 3, 1.0), lin["corr"], *m.export()])
        gone = m.evict((0.0, 0.0, 0.0), 60.0)
        got[-1] += [torch.tensor(gone), *m.knn(q, 3, 1.0), *m.export()]
        m.close()
    for a, b in zip(*got):
        assert torch.equal(a, b)
