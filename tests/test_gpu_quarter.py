"""Kernels that load the first quarter of each stage's twiddles and take the
second quarter from it, against the oracle bit for bit: inputs that make the
one exceptional entry count (the ratio of W^(L/4), cot(pi/2), is not minus
that of W^0: with zeros around, its tiny value or the sign of its zero reaches
the output), the inverse's tables, and the tables without the symmetry."""
import numpy as np
import pytest

import oracle
from paper_2604_00567_amd import binding, inputs
from tests.gpu_util import mismatches, run_gpu

pytestmark = pytest.mark.gpu

SIZES = [512, 1024, 2048, 4096, 8192, 1 << 14, 1 << 15, 1 << 16, 1 << 17, 1 << 20]
DTYPES = ["f16", "f32", "f16f32"]


def sparse(n, dtype, seed):
    """Three transforms that are zero (of both signs) but for a few values."""
    rng = np.random.default_rng(seed)
    x = np.zeros((3, n, 2), np.float32 if dtype == "f32" else np.float16)
    x[1] = -0.0
    for b in range(3):
        at = rng.choice(n, 4, replace=False)
        x[b, at, rng.integers(0, 2, 4)] = rng.uniform(-1, 1, 4)
    return x


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("n", SIZES)
def test_sparse_inputs(n, dtype):
    x = sparse(n, dtype, n % 1009)
    ref = oracle.emulate(x, "dual_select", dtype)
    single, cols, rows = binding.fft_config_count(n, dtype)
    print(f"sparse n={n} {dtype} variants={single}+{cols}x{rows}", flush=True)
    assert mismatches(run_gpu(x, dtype, "dual_select"), ref) == 0
    for v in range(single):
        assert mismatches(run_gpu(x, dtype, "dual_select", variant=(v, 0, False)), ref) == 0, v
    pairs = [(a % cols, a % rows) for a in range(max(cols, rows))] if cols and rows else []
    for a, b in pairs:
        assert mismatches(run_gpu(x, dtype, "dual_select", variant=(a, b, True)), ref) == 0, (a, b)


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("n", SIZES)
def test_inverse(n, dtype):
    import torch
    dense = inputs.uniform(n, 3, 41, "f32" if dtype == "f32" else "f16")
    for x in (sparse(n, dtype, 7), dense):
        xt = torch.from_numpy(x).to("cuda:0")
        yt = torch.empty_like(xt)
        plan = binding.Plan(n, 3, dtype, "dual_select", direction="inverse")
        plan.execute(xt, yt)
        torch.cuda.synchronize()
        print(f"inverse n={n} {plan.info()['config']}", flush=True)
        plan.close()
        assert mismatches(yt.cpu().numpy(), oracle.emulate(x, "dual_select", dtype, inverse=True)) == 0


@pytest.mark.parametrize("kind", ["linzer_feig", "cosine", "lf_w0_exempt"])
@pytest.mark.parametrize("n", [1024, 4096, 1 << 15, 1 << 18])
def test_other_tables(n, kind):
    x = inputs.uniform(n, 2, 43, "f32")
    assert mismatches(run_gpu(x, "f32", kind), oracle.emulate(x, kind, "f32")) == 0


@pytest.mark.parametrize("dtype,kind", [("f16", "dual_select"), ("f32", "dual_select"), ("f32", "linzer_feig")])
def test_uneven_batch_and_slot(dtype, kind):
    """Every size class once, sparse inputs, through an uneven batch (out of
    place) and a serving slot (in place)."""
    import torch
    sizes = [1 << m for m in range(1, 19)]
    off = np.concatenate([[0], np.cumsum(sizes)])
    x = np.concatenate([sparse(n, dtype, 90 + n % 83)[n.bit_length() % 3] if n > 2 else
                        np.full((n, 2), 0.5, np.float32 if dtype == "f32" else np.float16) for n in sizes])
    xt = torch.from_numpy(x).to("cuda:0")
    yt = torch.full_like(xt, float("nan"))
    batch = binding.Batch(sizes, dtype, kind)
    batch.execute(xt, yt)
    slot = binding.fft_serve_slot_create(dtype, kind, 1024, len(sizes), 8, 8 << 20)
    binding.fft_serve_slot_launch(slot, sizes, [1] * len(sizes), off[:-1], xt.data_ptr(),
                                  torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    binding.fft_serve_slot_destroy(slot)
    batch.close()
    for got in (yt.cpu().numpy(), xt.cpu().numpy()):
        for n, a in zip(sizes, off):
            ref = oracle.emulate(x[a:a + n][None], kind, dtype)
            assert mismatches(got[a:a + n][None], ref) == 0, n
