"""fft_plan_info describes the kernels that a plan launches: tables that hold the
quarter symmetry run that form, named in the text, with its LDS bytes (its copies
of the twiddles are shorter), the others the plain form of the same configuration."""
import re

import pytest

from paper_2604_00567_amd import binding

pytestmark = pytest.mark.gpu


def halves(n, batch, dtype, kind, direction="forward"):
    plan = binding.Plan(n, batch, dtype, kind, direction=direction)
    config = plan.info()["config"].split(" | ")
    plan.close()
    return [(re.sub(r",lds=\d+|,quarter", "", c), int(re.search(r"lds=(\d+)", c).group(1)), "quarter" in c)
            for c in config if "lds=" in c]


@pytest.mark.parametrize("n,batch,dtype", [(1 << 13, 4096, "f32"), (1 << 12, 16384, "f16"), (1 << 17, 512, "f16"),
                                           (1 << 16, 64, "f32")])
@pytest.mark.parametrize("direction", ["forward", "inverse"])
def test_quarter_form(n, batch, dtype, direction):
    quarter, plain = (halves(n, batch, dtype, kind, direction) for kind in ("dual_select", "linzer_feig"))
    assert len(quarter) == len(plain) == (2 if n >= 1 << 16 else 1)
    for q, p in zip(quarter, plain):
        assert q[0] == p[0]                      # one configuration
        assert q[2] and not p[2]
        assert q[1] < p[1]


def test_binary32_2e13_takes_four_workgroups_per_compute_unit():
    (_, lds, quarter), = halves(1 << 13, 4096, "f32", "dual_select")
    assert quarter and 160 * 1024 // lds == 4
