"""What the kept scratch chunks hold: a chunk serves every stream once its work
has ended."""
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
