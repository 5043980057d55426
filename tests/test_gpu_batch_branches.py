"""The uneven batch's graph on both sides of the line where its two list kernels
go into one branch (1.5 transforms of 2^16 points per compute unit), without
each of the lists, and replayed with eager work in between: every transform has
the bits of a plan of its size."""
import numpy as np
import pytest

from paper_2604_00567_amd import binding

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("more16,n15", [(0, 420), (1, 420), (0, 0), (-10 ** 6, 1100)])
def test_graph_matches_plans(more16, n15):
    import torch
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    n16 = max(0, 3 * cus // 2 + more16)
    counts = {16: n16, 15: n15, 14: 500, 10: 300, 6: 77}
    sizes = np.concatenate([np.full(c, 1 << m, dtype=np.int64) for m, c in counts.items()])
    total = int(sizes.sum())
    assert total > 1 << 25                     # replays a graph
    gen = torch.Generator(device="cuda").manual_seed(11)
    x = torch.rand((total, 2), device="cuda", generator=gen).sub_(0.5).half()
    y = torch.empty_like(x)
    b = binding.Batch(sizes, "f16", "dual_select")
    try:
        for _ in range(3):
            y.zero_()
            b.execute(x, y)
            torch.cuda.synchronize()
            at = 0
            for m, c in counts.items():
                if c == 0:
                    continue
                part = x[at:at + (c << m)]
                want = torch.empty_like(part)
                p = binding.Plan(1 << m, c, "f16", "dual_select")
                p.execute(part, want)
                torch.cuda.synchronize()
                p.close()
                assert torch.equal(y[at:at + (c << m)].view(torch.int16), want.view(torch.int16)), m
                at += c << m
    finally:
        b.close()
