"""What the kept scratch chunks hold: a chunk serves every stream once its work
has ended, and a release gives back what is idle at any time, without waiting."""
import threading

import pytest
import torch

from paper_2606_26010_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def far():
    from paper_2606_26010_amd import far as f
    f.lib()
    return f


def cloud(n, seed=1):
    g = synth.rng(seed)
    x = torch.from_numpy(g.uniform(-1, 1, (3, n)).astype("float32")).cuda()
    return x * torch.tensor([[60.0], [60.0], [3.0]], device="cuda")


def cov(far, x, stream=None):
    with torch.cuda.stream(stream or torch.cuda.default_stream()):
        return far.far_scan_covariances(x, 1.0, 5)


def test_a_null_stream_chunk_serves_other_streams(far):
    x = cloud(1200000)
    torch.cuda.synchronize()
    far.far_scratch_release()
    want = cov(far, x)
    torch.cuda.synchronize()
    held = far.far_scratch_reserved()
    for _ in range(2):
        got = cov(far, x, torch.cuda.Stream())
        torch.cuda.synchronize()
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
        assert far.far_scratch_reserved() == held


def test_release_does_not_wait_for_other_work(far):
    x = cloud(5000, 2)
    a = torch.randn(8192, 8192, device="cuda", dtype=torch.bfloat16)
    want = cov(far, x)
    torch.cuda.synchronize()
    held = far.far_scratch_reserved()
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        for _ in range(300):      # about 0.25 s
            a @ a
    far.far_scratch_release()
    assert not st.query()         # (the products are still running)
    assert far.far_scratch_reserved() < held
    torch.cuda.synchronize()
    got = cov(far, x)
    torch.cuda.synchronize()
    assert torch.equal(got[0], want[0])


@pytest.mark.parametrize("other_thread", [False, True])
def test_release_during_a_capture(far, other_thread):
    x, v = cloud(5000, 3), torch.arange(1000.0, device="cuda")
    cov(far, x), cov(far, x, torch.cuda.Stream())
    torch.cuda.synchronize()
    held = far.far_scratch_reserved()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        y = v * 2
        if other_thread:
            t = threading.Thread(target=far.far_scratch_release)
            t.start()
            t.join()
        else:
            far.far_scratch_release()
        y = y + 1
    assert far.far_scratch_reserved() < held
    for k in range(3):
        v.fill_(k)
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, torch.full_like(y, 2.0 * k + 1))


def test_a_small_call_leaves_the_large_chunk(far):
    x, s = cloud(1200000), cloud(5000, 4)
    t = torch.linspace(0, 0.1, 5000, device="cuda")
    vt = torch.linspace(-0.05, 0.15, 20, device="cuda", dtype=torch.float64)
    vel = torch.ones(20, 6, device="cuda", dtype=torch.float64)
    a = torch.randn(8192, 8192, device="cuda", dtype=torch.bfloat16)
    one, two = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    far.far_scratch_release()
    cov(far, x, one)
    torch.cuda.synchronize()
    held = far.far_scratch_reserved()
    with torch.cuda.stream(two):
        for _ in range(300):
            a @ a
        far.far_undistort(s, t, vt, vel)      # waits behind the products
    cov(far, x, one)
    assert not two.query()
    torch.cuda.synchronize()
    assert far.far_scratch_reserved() <= held + (64 << 20)


def test_a_request_the_device_cannot_hold(far):
    """Refused before anything runs, with what is idle given back, and no trace of
    it in the next call."""
    x = cloud(1200000)
    want = cov(far, x)
    cov(far, cloud(400000, 5), torch.cuda.Stream())
    torch.cuda.synchronize()
    assert far.far_scratch_reserved() > 0
    p = far.C.c_void_p(x.data_ptr())
    n = 1900000000                # 324 bytes of scratch each: 616 GB, the first request
    rc = far.lib().far_scan_covariances(p, n, 1.0, 5, p, p, None)
    assert rc == far.FAR_E_HIP and b"hipMallocFromPoolAsync" in far.lib().far_last_error()
    assert far.far_scratch_reserved() == 0
    got = cov(far, x)
    torch.cuda.synchronize()
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])


def test_held_memory_stays_bounded(far):
    """Large and small calls in turn on several streams without a host wait: at most
    the eight kept chunks and the caller's own."""
    sizes = [1200000, 5000, 400000, 32769]
    xs = [cloud(n, 10 + q) for q, n in enumerate(sizes)]
    torch.cuda.synchronize()
    far.far_scratch_release()
    cov(far, xs[0])
    torch.cuda.synchronize()
    big = far.far_scratch_reserved()
    streams = [torch.cuda.Stream() for _ in range(4)] + [torch.cuda.default_stream()]
    for r in range(60):
        cov(far, xs[(r * 7) % 4], streams[(r * 3) % 5])
    torch.cuda.synchronize()
    assert far.far_scratch_reserved() <= 9 * big
