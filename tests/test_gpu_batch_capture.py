"""Uneven batches in a stream capture, also those that eager calls replay as a graph of
their own: every replay has the bits of the eager call."""
import numpy as np
import pytest

from paper_2604_00567_amd import binding

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("more16,n15,n14", [(0, 60, 150), (1, 70, 100), (3, 40, 300), (150, 300, 100)])
@pytest.mark.parametrize("first", ["eager", "captured"])
def test_capture(more16, n15, n14, first):
    import torch
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    counts = {16: cus + more16, 15: n15, 14: n14, 6: 33}
    sizes = np.concatenate([np.full(c, 1 << m, dtype=np.int64) for m, c in counts.items()])
    total = int(sizes.sum())
    gen = torch.Generator(device="cuda").manual_seed(23)
    x, other = (torch.rand((total, 2), device="cuda", generator=gen).sub_(0.5).half() for _ in range(2))
    y, want = torch.empty_like(x), torch.empty_like(x)
    batch = binding.Batch(sizes, "f16")
    if first == "eager":
        batch.execute(x, want)
        torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        batch.execute(x, y)
    got = []
    for _ in range(3):
        y.fill_(float("nan"))
        batch.execute(other, want)
        graph.replay()
        torch.cuda.synchronize()
        got.append(y.clone())
    batch.execute(x, want)
    torch.cuda.synchronize()
    batch.close()
    for r in got:
        assert torch.equal(r.view(torch.int16), want.view(torch.int16))
