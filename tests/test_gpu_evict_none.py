"""An eviction that no point leaves by keeps the map as it is and costs a pass over
the voxels, not over the points."""
import statistics
import time

import numpy as np
import pytest
import torch

from paper_2606_26010_amd import synth

pytestmark = pytest.mark.gpu


def filled(far, n):
    """A map of n points spread one a square metre over a rolling surface."""
    g = synth.rng(n)
    x = g.uniform(0, n ** 0.5, (3, n))
    x[2] = 3 * np.sin(0.1 * x[0])
    m = far.Map(1.0, 20, -1.0, 2 * n, 2 * n, 5)
    m.insert(torch.from_numpy(x.astype(np.float32)).cuda())
    return m


def us(m):
    ts = []
    for _ in range(22):
        torch.cuda.synchronize()
        t = time.perf_counter()
        assert m.evict((0.0, 0.0, 0.0), 1e5) == 0
        ts.append(time.perf_counter() - t)
    return 1e6 * statistics.median(ts[2:])


def test_cost_and_map_of_an_eviction_of_nothing():
    from paper_2606_26010_amd import far
    small, large = filled(far, 1000), filled(far, 1000000)
    before, st = large.export(), large.stats()
    a, b = us(small), us(large)
    print(f"nothing evicted: {a:.0f} us at 1000 points, {b:.0f} us at 1000000")
    # 16 bytes a voxel written and read, about 20 MB in the large map: 10 us at a
    # rate well below a copy's, and as much again for two launches over the points
    assert b <= a + 20.0
    assert large.stats() == st
    for p, q in zip(before, large.export()):
        assert torch.equal(p, q)
    # and one voxel less is a rebuild
    key = np.floor(before[0][:, 0].cpu().numpy().astype(np.float64))
    far_off = np.array([key[0], key[1], key[2]]) + 0.5
    d = np.floor(before[0].cpu().numpy().astype(np.float64)) + 0.5
    r = np.sqrt(((d - far_off[:, None]) ** 2).sum(0))
    gone = int((r == r.max()).sum())
    assert large.evict(far_off, float(np.nextafter(r.max(), 0)) - 1e-6) == gone
    assert large.stats()["n_points"] == st["n_points"] - gone
    small.close()
    large.close()


def test_emptying_a_small_map():
    """One launch clears the voxels and the ghosts; the map then fills as a new one."""
    from paper_2606_26010_amd import far
    g = synth.rng(6)
    x = torch.from_numpy(g.uniform(0, 8, (3, 280)).astype(np.float32)).cuda()
    m = far.Map(1.0, 5, -1.0, 1000, 1000, 5)
    m.insert(x)
    want = m.export()
    all_, none = [], []
    for _ in range(32):
        torch.cuda.synchronize()
        t = time.perf_counter()
        assert m.evict((4.0, 4.0, 4.0), 1e5) == 0
        none.append(time.perf_counter() - t)
        torch.cuda.synchronize()
        t = time.perf_counter()
        assert m.evict((1e5, 0.0, 0.0), 1.0) == want[0].shape[1]
        all_.append(time.perf_counter() - t)
        assert m.stats()["n_points"] == m.stats()["n_voxels"] == 0
        assert int((m.knn(x, 3, 1.0)[0] >= 0).sum()) == 0
        m.insert(x)
        for p, q in zip(want, m.export()):
            assert torch.equal(p, q)
    a, b = (1e6 * statistics.median(t[2:]) for t in (all_, none))
    print(f"280 points: all evicted {a:.0f} us, none {b:.0f} us")
    assert a <= b + 20.0
    m.close()
