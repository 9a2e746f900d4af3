"""Scratch chunks wait for later calls: covariances enqueued on several streams
without a host wait, from several threads at once, with sizes that grow and
shrink around a chunk, on streams that end, and across releases of the scratch,
equal bit for bit what one call alone gives; and what is held stays bounded."""
import threading

import numpy as np
import pytest
import torch

from paper_2606_26010_amd import synth

pytestmark = pytest.mark.gpu

SIZES = [1, 300, 5000, 32769, 400000, 1200000]


@pytest.fixture(scope="module")
def scans():
    from paper_2606_26010_amd import far
    out = []
    for q, n in enumerate(SIZES):
        g = synth.rng(500 + q)
        span = np.array([[60.0], [60.0], [3.0]]) * max(n / 3e5, 0.2) ** 0.5
        x = torch.from_numpy((g.uniform(-1, 1, (3, n)) * span).astype(np.float32)).cuda()
        cov, val = far.far_scan_covariances(x, 1.0, 5)
        torch.cuda.synchronize()
        out.append((x, cov.clone(), val.clone()))
    return far, out


def same(got, want):
    return torch.equal(got[0], want[1]) and torch.equal(got[1], want[2])


def test_streams_without_a_host_wait(scans):
    far, sc = scans
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(3)]
    got = []
    for r in range(4):
        for q in [0, 5, 2, 4, 1, 3]:
            st = streams[(r + q) % 3]
            with torch.cuda.stream(st):
                got.append((q, far.far_scan_covariances(sc[q][0], 1.0, 5)))
        if r == 1:
            far.far_scratch_release()       # with calls still running
    torch.cuda.synchronize()
    for q, g in got:
        assert same(g, sc[q]), SIZES[q]


def test_threads_and_streams_that_end(scans):
    far, sc = scans
    torch.cuda.synchronize()
    bad, held = [], []

    def work(k):
        for r in range(6):
            q = (k + r) % len(SIZES)
            st = torch.cuda.Stream() if k % 2 else torch.cuda.default_stream()
            with torch.cuda.stream(st):
                g = far.far_scan_covariances(sc[q][0], 1.0, 5)
            st.synchronize()
            if not same(g, sc[q]):
                bad.append((k, r, SIZES[q]))

    for _ in range(2):
        th = [threading.Thread(target=work, args=(k,)) for k in range(6)]
        for t in th:
            t.start()
        for t in th:
            t.join()
        torch.cuda.synchronize()
        held.append(far.far_scratch_reserved())
    assert not bad, bad
    far.far_scratch_release()
    assert far.far_scratch_reserved() < max(held)
