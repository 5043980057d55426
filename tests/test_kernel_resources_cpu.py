"""Registers of the binary16 2^16-point kernels: 1024 lanes with 64 elements each have
128 registers a lane, and the forms that dual-select plans, uneven batches and
serving slots launch fit them, with nothing in scratch memory."""
import os
import re
import subprocess

import pytest

from paper_2604_00567_amd import build

UNIT = r"""
#include "batch_launch.hpp"
#include "fft_batch.hpp"
namespace dsfft {
template __global__ void fft_list_kernel<uint32_t, 16, 6, 6, 5, 5, 2048, ENC_QUARTER>(
    const uint32_t*, uint32_t*, const TwH*, const int64_t*, int64_t);
template __global__ void fft_list_kernel<uint32_t, 15, 5, 5, 5, 5, 1024, ENC_QUARTER>(
    const uint32_t*, uint32_t*, const TwH*, const int64_t*, int64_t);
#define PLAN(PIPE, ENC) \
    template __global__ void fft_unit_kernel<uint32_t, 16, 6, 1, 1, MODE_SMALL, 6, 5, 5, 0, 0, PIPE, uint32_t, uint32_t, ENC>( \
        const uint32_t*, uint32_t*, const TwH*, int64_t, int);
PLAN(0, ENC_QUARTER) PLAN(3, ENC_QUARTER) PLAN(0, ENC_QUARTER_INV) PLAN(3, ENC_QUARTER_INV)
}
"""


def test_no_scratch_memory(tmp_path):
    try:
        hipcc = build._hipcc()
    except RuntimeError:
        pytest.skip("no hipcc")
    src = tmp_path / "unit.hip"
    src.write_text(UNIT)
    r = subprocess.run([hipcc, "-x", "hip"] + build.COMMON + build.HIP_FLAGS +
                       ["-Rpass-analysis=kernel-resource-usage", "--cuda-device-only", "-c", str(src), "-o", os.devnull],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    names = re.findall(r"Function Name: (\S+)", r.stderr)
    scratch = [int(v) for v in re.findall(r"ScratchSize \[bytes/lane\]: (\d+)", r.stderr)]
    assert len(names) == len(scratch) == 6, r.stderr
    assert dict(zip(names, scratch)) == {n: 0 for n in names}
