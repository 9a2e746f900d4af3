"""The source packed by gather or by scatter: the same bits on either side of the
line, and a scan in random order no slower below a former line than above it."""
import statistics
import time

import numpy as np
import pytest
import torch

from paper_2606_26010_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def job():
    """A map and 524289 points in random order on its surface, the last of them not
    finite, which sorts last and adds nothing."""
    from paper_2606_26010_amd import far
    g = synth.rng(5)
    x = g.uniform(0, 200, (3, 524289))
    x[2] = 3 * np.sin(0.1 * x[0]) + g.normal(0, 0.02, x.shape[1])
    x = torch.from_numpy(x.astype(np.float32)).cuda()
    x[:, 131072] = x[:, 524288] = float("nan")
    m = far.Map(1.0, 20, -1.0, 1 << 20, 1 << 17, 5)
    m.insert(x[:, :400000].contiguous())
    cov, val = far.far_scan_covariances(x, 1.0, 5)
    T = np.eye(4)
    T[:3, 3] = (0.1, -0.05, 0.02)
    yield lambda n, p=0: m.linearize(x[:, :n].contiguous(), cov[:, :n].contiguous(),
                                     val[:n].contiguous(), T, 1.0, 0.5, precision=p,
                                     want_corr=True)
    m.close()


@pytest.mark.parametrize("prec", [0, 1])
def test_same_bits_on_both_sides(job, prec):
    a, b = job(131072, prec), job(131073, prec)
    assert torch.equal(a["corr"], b["corr"][:131072]) and int(b["corr"][131072]) == -1
    assert a["n_inliers"] == b["n_inliers"] > 100000
    np.testing.assert_array_equal(a["H"], b["H"])
    np.testing.assert_array_equal(a["b"], b["b"])
    assert a["cost"] == b["cost"]


def test_random_order_is_not_slower(job):
    def us(n):
        ts = []
        for _ in range(32):
            torch.cuda.synchronize()
            t = time.perf_counter()
            job(n)
            torch.cuda.synchronize()
            ts.append(time.perf_counter() - t)
        return 1e6 * statistics.median(ts[2:])

    a, b = us(524288), us(524289)
    print(f"524288 points in random order {a:.0f} us, 524289 {b:.0f} us")
    assert a <= b + 25.0
