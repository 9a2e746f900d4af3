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
