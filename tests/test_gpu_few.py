"""Calls of few transforms, bit for bit against the oracle: whole-transform
sizes split through the output (both directions, a table without the quarter
symmetry, in place, through fft_execute_scratch and in a replayed graph), at one
transform and on both sides of the limit; and the narrow column and row
kernels that two-pass plans of few transforms take."""
import numpy as np
import pytest

import oracle
from paper_2604_00567_amd import binding, inputs
from tests.gpu_util import mismatches

pytestmark = pytest.mark.gpu

SPLIT = [("f16", 14), ("f16", 15), ("f16", 16), ("f32", 13), ("f32", 14), ("f32", 15)]


def run(x, dtype, kind="dual_select", direction="forward", how="execute"):
    """(output, plan configuration); `x` tiled on the device if it is a (block, batch) pair."""
    import torch
    block, batch = x if isinstance(x, tuple) else (x, x.shape[0])
    xt = torch.from_numpy(block).to("cuda:0")
    xt = xt.repeat((batch + len(block) - 1) // len(block), 1, 1)[:batch].contiguous()
    yt = xt if how == "in_place" else torch.full_like(xt, float("nan"))
    plan = binding.Plan(block.shape[1], batch, dtype, kind, direction=direction)
    (plan.execute_scratch if how == "scratch" else plan.execute)(xt, yt)
    torch.cuda.synchronize()
    config = plan.info()["config"]
    plan.close()
    return yt, config


@pytest.mark.parametrize("dtype,log_n", SPLIT)
@pytest.mark.parametrize("direction", ["forward", "inverse"])
def test_split_sizes(dtype, log_n, direction):
    n = 1 << log_n
    x = inputs.uniform(n, 2, 50 + log_n, dtype)
    x[1] = 0                                     # few nonzero values, zeros of both signs
    x[1, :, 1] = -0.0
    x[1, [1, n // 3, n - 2], [0, 1, 0]] = [0.5, -0.25, 1.0]
    ref = oracle.emulate(x, "dual_select", dtype, inverse=direction == "inverse")
    splits = []
    for batch in (1, 2, 17, 48, 49, 97):
        y, config = run((x, batch), dtype, direction=direction)
        splits.append("split" in config)
        print(f"few n=2^{log_n} {dtype} {direction} batch={batch} {config}", flush=True)
        for b in {0, batch - 1, batch // 2, min(1, batch - 1)}:
            assert mismatches(y[b].cpu().numpy()[None], ref[b % 2][None]) == 0, (batch, b)
    assert splits[0] and not splits[-1]


@pytest.mark.parametrize("dtype,log_n", SPLIT)
def test_other_routes_give_the_same(dtype, log_n):
    x = inputs.uniform(1 << log_n, 3, 60 + log_n, dtype)
    ref = oracle.emulate(x, "dual_select", dtype)
    for how in ("in_place", "scratch"):
        assert mismatches(run(x, dtype, how=how)[0].cpu().numpy(), ref) == 0, how
    if dtype == "f32":                           # binary16 Linzer-Feig overflows
        y, config = run(x, dtype, kind="linzer_feig")
        assert "split" in config
        assert mismatches(y.cpu().numpy(), oracle.emulate(x, "linzer_feig", dtype)) == 0


def test_split_in_a_replayed_graph():
    import torch
    n = 1 << 15
    x = [inputs.uniform(n, 3, 70 + k, "f16") for k in range(3)]
    xt = torch.from_numpy(x[0]).to("cuda:0")
    yt, eager = torch.empty_like(xt), torch.empty_like(xt)
    plan = binding.Plan(n, 3, "f16", "dual_select")
    plan.execute(xt, yt)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        plan.execute(xt, yt)
    for k in (1, 2, 0):
        xt.copy_(torch.from_numpy(x[k]))
        plan.execute(xt, eager)                  # the program's own work between replays
        yt.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(yt.view(torch.int16), eager.view(torch.int16)), k
        assert mismatches(yt.cpu().numpy(), oracle.emulate(x[k], "dual_select", "f16")) == 0
    plan.close()


@pytest.mark.parametrize("dtype", ["f16", "f32", "f16f32"])
@pytest.mark.parametrize("log_n,batch", [(16, 4), (17, 1), (17, 9), (17, 32), (18, 2), (19, 1), (20, 1), (20, 3)])
def test_two_pass_plans_of_few_transforms(dtype, log_n, batch):
    x = inputs.uniform(1 << log_n, min(batch, 3), 80 + log_n, "f32" if dtype == "f32" else "f16")
    ref = oracle.emulate(x, "dual_select", dtype)
    y, config = run((x, batch), dtype)
    print(f"few n=2^{log_n} {dtype} batch={batch} {config}", flush=True)
    for b in {0, batch - 1, batch // 2}:
        assert mismatches(y[b].cpu().numpy()[None], ref[b % len(x)][None]) == 0, b


@pytest.mark.parametrize("short,long", [(3, 5), (49, 65), (97, 1)])
def test_lists_of_small_batches(short, long):
    """Binary16 batches below the graph's size: their 2^16 (`short`) and 2^15
    (`long`) transforms on both sides of the split limits, mixed with others,
    out of place, in place, and captured into a graph."""
    import torch
    rng = np.random.default_rng(short)
    sizes = np.array([1 << 16] * short + [1 << 15] * long + [1 << 17, 4096, 64, 2], np.int64)
    rng.shuffle(sizes)
    off = np.concatenate([[0], np.cumsum(sizes)])
    assert off[-1] <= 1 << 25
    blocks = {int(n): inputs.uniform(int(n), 3, 7, "f16") for n in set(sizes.tolist())}
    x = np.concatenate([blocks[int(n)][i % 3] for i, n in enumerate(sizes)])
    ref = {n: oracle.emulate(b, "dual_select", "f16") for n, b in blocks.items()}
    xt = torch.from_numpy(x).to("cuda:0")
    yt = torch.full_like(xt, float("nan"))
    batch = binding.Batch(sizes, "f16")
    batch.execute(xt, yt)
    zt = xt.clone()
    batch.execute(zt, zt)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    wt = torch.empty_like(xt)
    with torch.cuda.graph(graph):
        batch.execute(xt, wt)
    for _ in range(2):
        wt.fill_(float("nan"))
        batch.execute(xt, yt)
        graph.replay()
        torch.cuda.synchronize()
    batch.close()
    for got in (yt, zt, wt):
        y = got.cpu().numpy()
        for i, n in enumerate(sizes.tolist()):
            assert mismatches(y[off[i]:off[i + 1]][None], ref[n][i % 3][None]) == 0, (i, n)
