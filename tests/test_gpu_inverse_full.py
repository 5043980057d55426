"""The inverse kernels of the tuned configurations (several transforms, columns or
rows per workgroup), which small batches do not run: 2^26 elements of every size from
2^9 on, and two batches in between, against the oracle.  The input repeats three
transforms, so every transform of the output is compared, on the device, with the
three that the oracle checks."""
import pytest

import oracle
from paper_2604_00567_amd import binding, inputs
from tests.gpu_util import mismatches

pytestmark = pytest.mark.gpu

FULL = [(m, (1 << 26) >> m, d) for d in ("f16", "f32", "f16f32") for m in range(9, 21)]


@pytest.mark.parametrize("log_n,batch,dtype", FULL + [(18, 7, "f32"), (13, 1001, "f32"), (17, 65, "f16")])
def test_inverse_of_tuned_kernels(log_n, batch, dtype):
    import torch
    n = 1 << log_n
    plan = binding.Plan(n, batch, dtype, "dual_select", direction="inverse")
    config = plan.info()["config"]
    print(f"inverse n=2^{log_n} x {batch} {dtype} {config}", flush=True)
    if (log_n, batch, dtype) in FULL:
        tuned = binding.Plan(n, batch, dtype, "dual_select", variant=binding.fft_tuned_choice(n, dtype))
        assert config == tuned.info()["config"]
        tuned.close()
    x = inputs.uniform(n, 3, 17 + log_n, "f32" if dtype == "f32" else "f16")
    ref = oracle.emulate(x, "dual_select", dtype, inverse=True)
    xt = torch.from_numpy(x).to("cuda:0").repeat((batch + 2) // 3, 1, 1)[:batch].contiguous()
    yt = torch.full_like(xt, float("nan"))
    plan.execute(xt, yt)
    torch.cuda.synchronize()
    plan.close()
    assert mismatches(yt[:3].cpu().numpy(), ref[:min(3, batch)]) == 0
    bits = yt.view(torch.int16 if dtype != "f32" else torch.int32)
    assert torch.equal(bits[3:], bits[:-3])
