"""The relation that lets a kernel take the second quarter of a stage's twiddles
from the first, on the library's rounded tables: W_L^(j + L/4) is on the other
path, with the other sign of t and (sigma' m', m') = (m, -sigma m) (inverse:
(-m, sigma m)); dual-select tables hold it bit for bit for every j but the
ratio of j = 0, whose two values do not depend on L; the other tables do not."""
import numpy as np
import pytest

from paper_2604_00567_amd import binding


def quarters(n, dtype, kind, direction):
    m, t, path = binding.fft_table_build(n, dtype, kind, direction)
    sm = np.where(path == 1, -m, m)
    q = n // 4
    return [(a[:q], a[q:]) for a in (sm, m, t, path)]


def same(a, b):
    u = np.uint16 if a.dtype == np.float16 else np.uint32
    return a.view(u) == b.view(u)


@pytest.mark.parametrize("direction", ["forward", "inverse"])
@pytest.mark.parametrize("dtype", ["f16", "f32"])
def test_dual_select_holds_the_relation(dtype, direction):
    first = None
    for log_n in range(2, 21):
        (sm, smq), (m, mq), (t, tq), (p, pq) = quarters(1 << log_n, dtype, "dual_select", direction)
        s = 1 if direction == "forward" else -1
        assert np.all(pq != p), log_n
        assert np.all(same(smq, s * m)) and np.all(same(mq, -s * sm)), log_n
        assert np.all(same(tq[1:], -t[1:])), log_n
        ends = (t[:1], tq[:1])
        first = first or ends
        assert all(same(a, b) for a, b in zip(ends, first)), log_n


@pytest.mark.parametrize("kind", ["linzer_feig", "cosine", "lf_w0_exempt"])
def test_other_tables_do_not(kind):
    (_, _), (_, _), (_, _), (p, pq) = quarters(16, "f32", kind, "forward")
    assert not np.all(pq != p)


@pytest.mark.parametrize("log_l0", [2, 3, 4, 5, 6])
@pytest.mark.parametrize("lr", [1, 2, 3, 4, 5])
def test_copy_of_the_loaded_entries(log_l0, lr):
    """The LDS copy of a pass (span L0 before it, radix 2^lr): entry k of the copy
    comes from table entry k + L0 for k < L0, k + L0 2^floor(log2(k / L0))
    beyond; the pass reads entry q + L0 c at q + L0 slot(c) for the c that are
    loaded.  Both name the same table entries, each slot once, all of them below
    the copy's length.  (Row units: the same with L0 = 1 and a unit index.)"""
    l0, r = 1 << log_l0, 1 << lr
    n = l0 * r // 2
    source = [k + (l0 if k < l0 else l0 << ((k // l0).bit_length() - 1)) for k in range(n)]
    used = {}
    for c in range(1, r):
        top = 1 << (c.bit_length() - 1)
        if c > 1 and c & (top // 2):
            continue                              # taken from the first quarter
        slot = 0 if c == 1 else c - top // 2
        for q in range(l0):
            used[q + l0 * slot] = q + l0 * c
    assert sorted(used) == list(range(n))
    assert [used[k] for k in range(n)] == source
    rows = [1 if k == 0 else k + (1 << (k.bit_length() - 1)) for k in range(r // 2)]
    assert rows == [used[k * l0] // l0 for k in range(r // 2)]
