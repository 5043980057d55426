"""A tuning record of the user's (from fft_tune, or a DSFFT_TUNE_FILE) decides the
kernels of later plans of as many transforms and more, also where they are few;
shipped records, and those tuned with more transforms, give way there to the shapes
for few transforms."""
import json
import os
import subprocess
import sys

import pytest

from paper_2604_00567_amd import binding

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
# log2 n, transforms, recorded variant: column and row kernels wider than a call of
# few transforms takes, and a whole transform where it would be split or on more lanes
RECORDS = [(18, 4, (1, 1, True)), (17, 1, (1, 1, True)), (16, 3, (0, 0, False)), (15, 100, (2, 0, False))]

PROGRAM = """
import json, sys
sys.path.insert(0, {root!r})
from paper_2604_00567_amd import binding
out = []
for log_n, batch, variant in {records!r}:
    recorded, given = binding.Plan(1 << log_n, batch, "f16"), binding.Plan(1 << log_n, batch, "f16", variant=variant)
    out.append([recorded.info()["config"], given.info()["config"]])
print(json.dumps(out))
"""


@pytest.mark.parametrize("tuned_batch", [None, 1, 1 << 16])
def test_record_file(tmp_path, tuned_batch):
    import torch
    props = torch.cuda.get_device_properties(0)
    tag = f"{props.gcnArchName.split(':')[0]} {props.multi_processor_count}"
    path = tmp_path / "records.txt"
    note = f"# batch {tuned_batch}\n" if tuned_batch else ""
    path.write_text("".join(f"{note}{tag} 0 {m} {a} {b} {int(two)} 1000.0\n" for m, _, (a, b, two) in RECORDS))
    r = subprocess.run([sys.executable, "-c", PROGRAM.format(root=ROOT, records=RECORDS)], capture_output=True, text=True,
                       env=dict(os.environ, DSFFT_TUNE_FILE=str(path)), timeout=100)
    assert r.returncode == 0, r.stderr
    for (recorded, given), record in zip(json.loads(r.stdout.splitlines()[-1]), RECORDS):
        assert (recorded == given) == (tuned_batch != 1 << 16), record


def test_tuned_in_this_process():
    n, batch = 1 << 19, 2
    before = binding.Plan(n, batch, "f16")
    assert "upw=32" not in before.info()["config"].split(" | ")[0]     # the shape for few transforms
    before.close()
    binding.fft_tune(n, batch, "f16", "dual_select", reps=2)
    a, b, two = binding.fft_tuned_choice(n, "f16")
    tuned, given = binding.Plan(n, batch, "f16"), binding.Plan(n, batch, "f16", variant=(a, b, two))
    assert tuned.info()["config"] == given.info()["config"]
    tuned.close()
    given.close()
