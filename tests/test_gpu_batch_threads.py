"""Two threads that execute one batch on one stream, each on its own buffers: every
call transforms the buffers it was given, in batches that replay a graph (whose
nodes each call points at its buffers) and in batches launched in order."""
import threading

import numpy as np
import pytest

from paper_2604_00567_amd import binding

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("count16,count10", [(500, 2000), (20, 3000)])
def test_threads_share_a_batch(count16, count10):
    import torch
    sizes = np.array([1 << 16] * count16 + [1 << 10] * count10, np.int64)
    total = int(sizes.sum())
    assert (total > 1 << 25) == (count16 == 500)
    gen = torch.Generator(device="cuda").manual_seed(5)
    stream = torch.cuda.Stream()
    batch = binding.Batch(sizes, "f16")
    calls, outs, wants, errors = 12, [], [], []
    with torch.cuda.stream(stream):
        xs = [torch.rand((total, 2), device="cuda", generator=gen).sub_(0.5).half() for _ in range(2)]
        for x in xs:
            outs.append([torch.full_like(x, float("nan")) for _ in range(calls)])
            wants.append(torch.empty_like(x))
            batch.execute(x, wants[-1])
    stream.synchronize()

    start = threading.Barrier(2)

    def run(x, ys):
        try:
            start.wait()
            for y in ys:
                batch.execute(x, y, stream=stream)
        except Exception as e:                      # noqa: BLE001 - reported by the test below
            errors.append(e)

    threads = [threading.Thread(target=run, args=a) for a in zip(xs, outs)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    stream.synchronize()
    batch.close()
    assert not errors
    for ys, want in zip(outs, wants):
        for k, y in enumerate(ys):
            assert torch.equal(y.view(torch.int16), want.view(torch.int16)), k
