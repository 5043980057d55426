"""Work lists of a serving slot at the edges of the kernel that copies them to the
device (16 bytes a lane, 256 lanes a block): lists that end inside a chunk, short
of one block, just past one, many blocks, and slots filled to their capacity.
Each step has the bits of plans of the same sizes."""
import numpy as np
import pytest

from paper_2604_00567_amd import binding, inputs
from tests.gpu_util import mismatches, run_gpu

pytestmark = pytest.mark.gpu

# dtype, (log2 n, transforms), work items, offsets: 48 bytes an item and 8 an
# offset, so an odd number of offsets ends inside a chunk; binary16 2^15 and 2^16
# are offsets only, a split 2^17 / 2^18 takes 16 / 32 items and no offset
STEPS = [
    ("f16", [(4, 1)], 1, 1),
    ("f16", [(16, 1)], 0, 1),
    ("f16", [(14, 77)], 77, 77),                     # 4312 bytes: 16 lanes past one block
    ("f16", [(18, 3), (15, 5), (17, 2), (8, 33)], 130, 38),
    ("f16", [(18, 40), (10, 17), (16, 3)], 1282, 20),
    ("f32", [(17, 3), (14, 2), (2, 5)], None, 7),
]


@pytest.mark.parametrize("dtype,reqs,items,offsets", STEPS)
def test_step_matches_plans(dtype, reqs, items, offsets):
    import torch
    n = np.array([1 << m for m, _ in reqs], dtype=np.int64)
    b = np.array([c for _, c in reqs], dtype=np.int64)
    off = np.concatenate([[0], np.cumsum(n * b)[:-1]])
    parts = [inputs.normal(int(v), int(c), 31 + i, dtype) for i, (v, c) in enumerate(zip(n, b))]
    flat = torch.from_numpy(np.concatenate([p.reshape(-1, 2) for p in parts])).to("cuda:0")
    wants = [run_gpu(p, dtype, "dual_select") for p in parts]
    data = torch.empty_like(flat)
    cap = 4096 if items is None else max(1, items)
    slot = binding.fft_serve_slot_create(dtype, "dual_select", cap, offsets, int(b.sum()),
                                         int((n * b).sum()) * (4 if dtype == "f16" else 8))
    try:
        for _ in range(3):                     # later steps reuse the slot's buffers
            data.copy_(flat)
            binding.fft_serve_slot_launch(slot, n, b, off, data.data_ptr(), torch.cuda.current_stream().cuda_stream)
            torch.cuda.synchronize()
            out = data.cpu().numpy()
            for p, v, c, o, want in zip(parts, n, b, off, wants):
                assert mismatches(out[o:o + v * c].reshape(p.shape), want) == 0, (v, c)
    finally:
        binding.fft_serve_slot_destroy(slot)
