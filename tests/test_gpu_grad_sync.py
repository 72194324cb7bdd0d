"""wcl_grad synchronises the stream, as its declaration says."""
import pytest

from gpu_util import setup, to_gpu
from paper_1612_06556_amd import synth

pytestmark = pytest.mark.gpu


def test_nothing_is_pending_after_the_gradient():
    """The stream has nothing left to do when the call returns, every time (the
    kernel that reports dL/dkappa ends after the host has seen its value)."""
    import torch
    dims = (8, 8, 8, 8)
    lat, _, _ = setup(dims, -1, 0.12, 1.0, 1001, None)
    x, y = (to_gpu(synth.gaussian_spinor(dims, s)) for s in (94, 95))
    stream = torch.cuda.Stream()
    done = []
    with torch.cuda.stream(stream):
        for _ in range(200):
            lat.grad(x, y)
            done.append(stream.query())
    lat._sync_stream()
    assert all(done), done.count(False)
