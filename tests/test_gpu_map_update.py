"""Map updates at the sizes where their kernels change over, against the
oracle: covariances of added points on either side of the neighbour count up
to which they come from the certificates' search, insert sizes around a
block, and correspondences after each update."""
import math

import numpy as np
import pytest
import torch

from paper_2606_26010_amd import synth

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def host(t):
    return t.detach().cpu().numpy()


@pytest.mark.parametrize("k", [1, 9, 10, 11, 32])
def test_insert_covariances_by_neighbour_count(orc, k):
    from paper_2606_26010_amd import far
    gm = far.Map(1.0, 20, -1.0, 1 << 14, 0, k)
    om = orc.Map(1.0, 20, 1.0 / math.sqrt(20.0), k, point_capacity=1 << 14,
                 voxel_capacity=1 << 14)
    for seed, n in ((1, 1), (2, 255), (3, 257), (4, 4000), (5, 2)):
        b = synth.random_cloud(seed, n, extent=2.5, dup_frac=0.05, on_faces=0.1)
        assert gm.insert(dev(b)) == om.insert(b, check=False)[:2], n
        gx, gc, gv = gm.export()
        ox, oc, ov = om.export()
        np.testing.assert_array_equal(host(gx), ox)
        np.testing.assert_array_equal(host(gv), ov)
        np.testing.assert_allclose(host(gc), oc, rtol=2e-6, atol=1e-6)
        q = synth.random_cloud(seed + 50, 600, extent=4.0)
        cov, val = np.zeros((6, 600), np.float32), np.zeros(600, np.uint8)
        o = om.linearize(q, cov, val, np.eye(4), 1.0, 0.1, want_corr=True)
        g = gm.linearize(dev(q), dev(cov), dev(val), np.eye(4), 1.0, 0.1, want_corr=True)
        np.testing.assert_array_equal(host(g["corr"]), o["corr"])
    s = gm.stats()
    assert s["n_voxels"] == om.n_voxels and 1.0 <= s["mean_probe"] <= s["max_probe"]
    gm.close()


@pytest.mark.parametrize("n", [1, 255, 256, 257, 1024, 1025, 65536, 65537, 262145, 530001])
def test_downsample_and_insert_around_tile_sizes(n):
    """Sizes on both sides of the tiles of the flag scan and of the radix sort,
    against numpy's first occurrences (a map of one point per voxel and no
    spacing accepts the first point of every voxel)."""
    from paper_2606_26010_amd import far
    g = np.random.default_rng(n)
    x = (g.uniform(-1, 1, (3, n)) * np.array([[60.0], [8.0], [3.0]])).astype(np.float32)
    x[0, g.integers(0, n, n // 50)] = np.nan
    v = 0.5
    ok = np.isfinite(x).all(0)
    key = np.floor(x.astype(np.float64) / v)
    key[:, ~ok] = np.inf
    _, first = np.unique(key, axis=1, return_index=True)
    first = np.sort(first)
    first = first[ok[first]]
    pts, keep = far.far_voxel_downsample(dev(x), v, want_keep=True)
    np.testing.assert_array_equal(host(keep), first)
    np.testing.assert_array_equal(host(pts), x[:, first])
    m = far.Map(v, 1, 0.0, max(first.size, 1), 0, 1)
    assert m.insert(dev(x)) == (far.FAR_OK, first.size)
    np.testing.assert_array_equal(host(m.export()[0]), x[:, first])
    m.close()


def test_insert_refused_on_voxel_capacity_leaves_the_map(orc):
    """A batch whose new voxels do not fit changes nothing: the same map and the
    same answers after it, and a smaller batch then goes in as in the oracle."""
    from paper_2606_26010_amd import far
    gm = far.Map(1.0, 20, -1.0, 1 << 14, 200, 5)
    om = orc.Map(1.0, 20, 1.0 / math.sqrt(20.0), 5, point_capacity=1 << 14, voxel_capacity=200)
    for seed, ext in ((1, 2.5), (2, 30.0), (3, 2.5)):
        b = synth.random_cloud(seed, 2000, extent=ext)
        assert gm.insert(dev(b)) == om.insert(b, check=False)[:2], ext
        for a, o in zip(gm.export(), om.export()):
            np.testing.assert_allclose(host(a), o, rtol=2e-6, atol=1e-6)
        q = synth.random_cloud(9, 500, extent=4.0)
        np.testing.assert_array_equal(host(gm.knn(dev(q), 5, 1.0)[0]), om.knn(q, 5, 1.0)[0])
    gm.close()


@pytest.mark.parametrize("k,nmax", [(5, 2), (5, 64), (9, 20), (10, 64), (11, 20)])
def test_certificates_by_one_lane_and_by_four(k, nmax):
    """The same points (a crowded part, duplicates, a thin part) inserted alone
    and with so many far ones that one lane takes a point, then with those
    evicted: covariances and six iterations agree bit for bit."""
    from paper_2606_26010_amd import far
    a = synth.random_cloud(11, 3000, extent=1.5, dup_frac=0.05, on_faces=0.1)
    b = synth.random_cloud(12, 4001, extent=12.0, dup_frac=0.01)
    near = np.concatenate([a, b], 1)
    g = synth.rng(13)
    away = (g.uniform(-40.0, 40.0, (3, 60000)) + np.array([[500.0], [0.0], [0.0]])).astype(np.float32)
    q = dev((np.concatenate([a, b[:, :2000]], 1) + g.normal(scale=0.05, size=(3, 5000))).astype(np.float32))
    T = synth.random_offset(synth.rng(14), 0.05, 0.5)
    cov, val = far.far_scan_covariances(q, 1.0, 5)
    prm = far.align_params(1.0, 0.1, max_iters=6, eps=0.0)

    def state(m):
        x, c, v = m.export()
        _, Tg, st = m.align(q, cov, val, T, prm)
        ref = m.linearize(q, cov, val, T, 1.0, 0.1, want_corr=True)
        return [host(t)[..., :held] for t in (x, c, v)] + [np.asarray(Tg), host(ref["corr"])]

    def new(p):
        m = far.Map(1.0, nmax, 0.0, 1 << 17, 0, k)
        m.insert(dev(p))
        return m

    alone = new(near)
    held = alone.export()[0].shape[1]
    want = state(alone)
    both = new(np.concatenate([near, away], 1))
    for u, w in zip(want, state(both)):
        np.testing.assert_array_equal(u, w)
    assert both.evict([0.0, 0.0, 0.0], 100.0) > 0
    for u, w in zip(want, state(both)):
        np.testing.assert_array_equal(u, w)
