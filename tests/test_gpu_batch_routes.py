"""Uneven batches on both sides of the lines between launches in order and graphs
(below 2^25 elements too, where the 2^16-point list ends in a short round), out of
place, in place and on new buffers: every transform has the bits of a plan of its size."""
import numpy as np
import pytest

from paper_2604_00567_amd import binding

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rounds16,more16,n15,n14", [
    (1, 0, 60, 150),                 # one round: in order
    (1, 1, 0, 1),                    # a second round, nothing to fill it: in order
    (1, 1, 70, 100),                 # branches below 2^25 elements
    (1, 3, 40, 500),                 # lists in one branch
])
def test_batch_matches_plans(rounds16, more16, n15, n14):
    import torch
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    counts = {16: rounds16 * cus + more16, 15: n15, 14: n14, 6: 33}
    sizes = np.concatenate([np.full(c, 1 << m, dtype=np.int64) for m, c in counts.items()])
    total = int(sizes.sum())
    gen = torch.Generator(device="cuda").manual_seed(17)
    xs = [torch.rand((total, 2), device="cuda", generator=gen).sub_(0.5).half() for _ in range(2)]
    wants = []
    for x in xs:
        want, at = torch.empty_like(x), 0
        for m, c in counts.items():
            if c:
                p = binding.Plan(1 << m, c, "f16")
                p.execute(x[at:at + (c << m)], want[at:at + (c << m)])
                torch.cuda.synchronize()
                p.close()
            at += c << m
        wants.append(want)
    batch = binding.Batch(sizes, "f16")
    try:
        outs = [torch.full_like(x, float("nan")) for x in xs] + [x.clone() for x in xs]
        for k, y in enumerate(outs):
            batch.execute(xs[k] if k < 2 else y, y)
        torch.cuda.synchronize()
    finally:
        batch.close()
    for k, y in enumerate(outs):
        assert torch.equal(y.view(torch.int16), wants[k % 2].view(torch.int16)), k
