"""Two-pass plans of few transforms in place: columns and rows of one width, at one
transform, at the edges between the widths and past them (where the plan's own pair
runs), bit for bit against the oracle; and column launches on both sides of the
size up to which blocks of whole lines keep their plain order."""
import numpy as np
import pytest

import oracle
from paper_2604_00567_amd import binding, inputs
from tests.gpu_util import mismatches

pytestmark = pytest.mark.gpu


def check(plan, dtype, log_n, batch, direction, in_place):
    import torch
    x = inputs.uniform(1 << log_n, min(batch, 3), 80 + log_n, "f32" if dtype == "f32" else "f16")
    ref = oracle.emulate(x, "dual_select", dtype, inverse=direction == "inverse")
    xt = torch.from_numpy(x).to("cuda:0").repeat((batch + 2) // 3, 1, 1)[:batch].contiguous()
    yt = xt if in_place else torch.full_like(xt, float("nan"))
    plan.execute(xt, yt)
    torch.cuda.synchronize()
    for b in {0, batch - 1, batch // 2, min(1, batch - 1)}:
        assert mismatches(yt[b].cpu().numpy()[None], ref[b % len(x)][None]) == 0, b


# units per workgroup in place on 256 compute units (None: the plan's own pair)
@pytest.mark.parametrize("dtype,log_n,batch,width", [
    ("f16", 17, 1, 16), ("f16", 17, 8, 16), ("f16", 17, 9, 32), ("f16", 17, 32, 32), ("f16", 17, 33, 64),
    ("f16", 17, 64, 64), ("f16", 17, 65, None), ("f16", 18, 3, 16), ("f16", 20, 7, 32),
    ("f32", 16, 8, None), ("f32", 17, 7, 16), ("f32", 17, 14, 16), ("f32", 17, 18, None), ("f32", 18, 2, None),
    ("f16f32", 16, 24, 32), ("f16f32", 17, 4, None), ("f16f32", 17, 8, 16), ("f16f32", 18, 1, None),
])
@pytest.mark.parametrize("direction", ["forward", "inverse"])
def test_in_place(dtype, log_n, batch, width, direction):
    import torch
    plan = binding.Plan(1 << log_n, batch, dtype, direction=direction)
    try:
        config = plan.info()["config"]
        print(f"in place n=2^{log_n} {dtype} {direction} batch={batch} {config}", flush=True)
        if torch.cuda.get_device_properties(0).multi_processor_count == 256:
            assert ("in place" in config) == (width is not None), config
            assert width is None or f"in place: {width} columns" in config, config
        check(plan, dtype, log_n, batch, direction, True)
        check(plan, dtype, log_n, batch, direction, False)
    finally:
        plan.close()


@pytest.mark.parametrize("dtype,log_n,batch,columns", [
    ("f16", 17, 32, 32), ("f16", 17, 33, 32), ("f16", 17, 70, 64), ("f32", 18, 8, 16), ("f32", 18, 9, 16),
    ("f16f32", 17, 40, 32),
])
def test_order_of_whole_line_columns(dtype, log_n, batch, columns):
    _, cols, rows = binding.fft_config_count(1 << log_n, dtype)
    ran = 0
    for a in range(cols):
        plan = binding.Plan(1 << log_n, batch, dtype, variant=(a, a % rows, True))
        if f"upw={columns}," in plan.info()["config"].split(" | ")[0]:
            check(plan, dtype, log_n, batch, "forward", False)
            check(plan, dtype, log_n, batch, "forward", True)
            ran += 1
        plan.close()
    assert ran
