"""Downsampling scans of few voxels: the first point of each, whatever the order, in
a time that crowding does not multiply."""
import statistics
import time

import numpy as np
import pytest
import torch

from paper_2606_26010_amd import synth

pytestmark = pytest.mark.gpu


def scan(n, voxels, in_order):
    g = synth.rng(n + voxels)
    x = g.uniform(0, 1, (3, n))
    x[0] = np.floor(g.uniform(0, voxels, n)) + 0.99 * x[0]
    if in_order:
        x = x[:, np.argsort(np.floor(x[0]), kind="stable")]
    return np.ascontiguousarray(x.astype(np.float32))


@pytest.mark.parametrize("in_order", [False, True])
@pytest.mark.parametrize("voxels", [1, 3, 10, 100])
@pytest.mark.parametrize("n", [1, 63, 64, 65, 257, 5000, 100000])
def test_first_points(n, voxels, in_order):
    from paper_2606_26010_amd import far
    x = scan(n, voxels, in_order)
    x[n % 3, 7::29] = np.nan
    pts, keep = far.far_voxel_downsample(torch.from_numpy(x).cuda(), 1.0, want_keep=True)
    ok = np.flatnonzero(np.isfinite(x).all(0))
    _, first = np.unique(np.floor(x[0, ok]), return_index=True)
    want = np.sort(ok[first])
    np.testing.assert_array_equal(keep.cpu().numpy(), want)
    np.testing.assert_array_equal(pts.cpu().numpy(), x[:, want])


def test_one_voxel_is_not_much_slower_than_many():
    from paper_2606_26010_amd import far

    def us(voxels):
        x = torch.from_numpy(scan(1000000, voxels, False)).cuda()
        ts = []
        for _ in range(12):
            torch.cuda.synchronize()
            t = time.perf_counter()
            far.far_voxel_downsample(x, 1.0)
            torch.cuda.synchronize()
            ts.append(time.perf_counter() - t)
        return 1e6 * statistics.median(ts[2:])

    one, many = us(1), us(1000)
    print(f"1000000 points in one voxel {one:.0f} us, in 1000 voxels {many:.0f} us")
    assert one <= 2.5 * many


def test_thirty_voxels_in_random_order():
    """Where the lanes of a wave meet by twos: no slower than a few times the scan of
    many voxels."""
    from paper_2606_26010_amd import far

    def us(voxels):
        x = torch.from_numpy(scan(1000000, voxels, False)).cuda()
        ts = []
        for _ in range(12):
            torch.cuda.synchronize()
            t = time.perf_counter()
            far.far_voxel_downsample(x, 1.0)
            torch.cuda.synchronize()
            ts.append(time.perf_counter() - t)
        return 1e6 * statistics.median(ts[2:])

    few, many = us(21), us(1000)
    print(f"1000000 points in 21 voxels {few:.0f} us, in 1000 {many:.0f} us")
    assert few <= 3.0 * many
