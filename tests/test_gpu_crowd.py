"""Crowded scans: below the points of the wide covariances, which deal a cell to 32
lanes, the call still takes one lane per point where the cells are full.  Either
search gives the same bits, and the call is never far slower than the latter."""
import statistics
import time

import numpy as np
import pytest
import torch

from paper_2606_26010_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def far():
    from paper_2606_26010_amd import far as f
    f.lib()
    return f


def scan(kind, n, per_cell, stray=False):
    g = synth.rng(n + per_cell)
    d = 2 if kind == "plane" else 3
    x = g.uniform(0, (n / per_cell) ** (1.0 / d), (3, n))
    if d == 2:
        x[2] = 0.5 + g.normal(0, 0.01, n)
    if stray:                     # a wide key range, and points without a key
        x[:, ::97] += g.uniform(-300, 300, (3, x[:, ::97].shape[1]))
        x[0, 5::211] = np.nan
    return torch.from_numpy(x.astype(np.float32)).cuda()


def us(f):
    """Median time of 10 calls, each waited for."""
    ts = []
    for _ in range(12):
        torch.cuda.synchronize()
        t = time.perf_counter()
        f()
        torch.cuda.synchronize()
        ts.append(time.perf_counter() - t)
    return 1e6 * statistics.median(ts[2:])


def one_lane(far, f):
    far.far_set_covariance_schedule(1 << 30)   # no run is that long: no wave per run
    try:
        return f()
    finally:
        far.far_set_covariance_schedule(0)


@pytest.mark.parametrize("kind", ["plane", "heap"])
@pytest.mark.parametrize("n,per_cell", [(512, 300), (513, 600), (2000, 150), (2000, 1000),
                                        (9000, 9000), (28672, 10), (28672, 43), (28672, 2000)])
def test_same_bits_on_either_side_of_the_lines(far, kind, n, per_cell):
    for stray in (False, True):
        x = scan(kind, n, per_cell, stray)
        for k in (4, 5, 10):
            a = far.far_scan_covariances(x, 1.0, k)
            b = one_lane(far, lambda: far.far_scan_covariances(x, 1.0, k))
            assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1]), (stray, k)
    offs = torch.tensor([0, n // 3, n // 3, n], device="cuda")
    a = far.far_scan_covariances_batch(x, offs, 1.0, 5)
    b = one_lane(far, lambda: far.far_scan_covariances_batch(x, offs, 1.0, 5))
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])


@pytest.mark.parametrize("n,per_cell", [(8000, 1000), (16000, 1000), (28000, 300),
                                        (28000, 28000)])
def test_crowded_scans_are_not_slower(far, n, per_cell):
    x = scan("plane", n, per_cell)
    call = us(lambda: far.far_scan_covariances(x, 1.0, 5))
    lane = one_lane(far, lambda: us(lambda: far.far_scan_covariances(x, 1.0, 5)))
    print(f"{n} points, {per_cell} a cell: {call:.0f} us, one lane per point {lane:.0f} us")
    assert call <= 1.3 * lane


def test_scans_of_a_batch_do_not_crowd_each_other(far):
    """One scan many times over: its copies share cells, but not their points."""
    one = scan("heap", 300, 20)
    x = one.repeat(1, 20)
    offs = torch.arange(21, device="cuda") * 300
    want = far.far_scan_covariances(one, 1.0, 5)
    got = far.far_scan_covariances_batch(x, offs, 1.0, 5)
    assert torch.equal(got[0], want[0].repeat(1, 20)) and torch.equal(got[1], want[1].repeat(20))
    wide = us(lambda: far.far_scan_covariances_batch(x, offs, 1.0, 5))
    lane = one_lane(far, lambda: us(lambda: far.far_scan_covariances_batch(x, offs, 1.0, 5)))
    print(f"20 scans of 300 points: {wide:.0f} us, one lane per point {lane:.0f} us")
    assert wide < lane


def line(n, length):
    """n points along x over length cells."""
    g = synth.rng(n + length)
    x = np.full((3, n), 0.25)
    x[0] = g.uniform(0, length, n)
    x[1:] += g.uniform(0, 1e-3, (2, n))
    return torch.from_numpy(x.astype(np.float32)).cuda()


def test_a_long_run_costs_no_more_than_short_ones(far):
    """Points in one cell and along 600 cells, with two far ones that give the sort 15
    bits of x below the cell: few candidates each, so about the same time."""
    one, many = line(600000, 1), line(600000, 600)
    one[0, :2] = many[0, :2] = torch.tensor([-2000.0, 2000.0])
    a = us(lambda: far.far_scan_covariances(one, 1.0, 1))
    b = us(lambda: far.far_scan_covariances(many, 1.0, 1))
    print(f"600000 points in one cell {a:.0f} us, in 600 cells {b:.0f} us")
    assert a <= 1.5 * b


@pytest.mark.parametrize("n", [1023, 1024, 1025, 1026, 1027, 2560, 9999])
def test_long_runs_against_the_oracle(far, orc, n):
    """Runs around the length that a wave labels, from every offset of the sorted
    order, between short ones."""
    g = synth.rng(n)
    x = line(n, 1).cpu().numpy()
    for before in range(4):
        few = (g.uniform(0, 1, (3, before)) - np.array([[3.0], [0.0], [0.0]])).astype(np.float32)
        more = (g.uniform(0, 2, (3, 40)) + np.array([[1.0], [0.0], [0.0]])).astype(np.float32)
        p = np.ascontiguousarray(np.concatenate([few, x, more], 1))
        cov, val = far.far_scan_covariances(torch.from_numpy(p).cuda(), 1.0, 5)
        oc, ov = orc.scan_covariances(p, 1.0, 5)
        np.testing.assert_array_equal(val.cpu().numpy(), ov)
        np.testing.assert_allclose(cov.cpu().numpy(), oc, rtol=2e-6, atol=1e-6)
