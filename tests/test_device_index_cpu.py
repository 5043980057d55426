"""The index functions of the device code, compiled for the host: the order of the
column kernels' blocks, the slots of the LDS copies that hold only the loaded
twiddles, and the places of the two-pass intermediate in the output."""
import subprocess

import pytest

from paper_2604_00567_amd import build

PROGRAM = r"""
#include <cstdio>
#include <set>
#include <vector>
#include "fft_device.hpp"
#include "tables.hpp"
using namespace dsfft;

static int bad = 0;
#define EXPECT(c) do { if (!(c)) { if (bad++ < 20) std::printf("line %d: %s\n", __LINE__, #c); } } while (0)

// blocks 0 .. n-1 exactly once; whole-line blocks of small launches in place
template <bool LINES> static void order(int64_t n, int64_t bytes) {
    std::vector<char> seen(n, 0);
    for (int64_t b = 0; b < n; ++b) {
        const int64_t c = column_block<LINES>(b, n, bytes);
        EXPECT(c >= 0 && c < n && !seen[c]);
        if (c >= 0 && c < n) seen[c] = 1;
        if (LINES && bytes <= kPlainOrderBytes) EXPECT(c == b);
        // an XCD (b % 8) takes runs of consecutive blocks
        if (n >= 8 * kColumnRun && b < 8 * kColumnRun && !(LINES && bytes <= kPlainOrderBytes))
            EXPECT(c / kColumnRun == b % 8);
    }
}

// A pass of span L0 and radix R: the entries that are loaded (quarter_loads) have one
// slot each, below the copy's length, no two the same.
template <int LOG_L0, int LR> static void slots() {
    constexpr int L0 = 1 << LOG_L0, R = 1 << LR;
    std::set<int> used, row;
    for (int c = 1; c < R; ++c) {
        if (!quarter_loads(ENC_QUARTER, c)) continue;
        EXPECT(row.insert(row_slot(ENC_QUARTER, c)).second);
        for (int q = 0; q < L0; ++q) EXPECT(used.insert(q + L0 * quarter_slot(c)).second);
    }
    EXPECT((int)used.size() == L0 * R / 2 && *used.begin() == 0 && *used.rbegin() == L0 * R / 2 - 1);
    EXPECT((int)row.size() == R / 2 && *row.rbegin() == R / 2 - 1);
    // what the copy loops put there: table entry k + L0 2^floor(log2(k / L0))
    for (int c = 1; c < R; ++c) {
        if (!quarter_loads(ENC_QUARTER, c)) continue;
        for (int q = 0; q < L0; ++q) {
            const int k = q + L0 * quarter_slot(c);
            const unsigned h = (unsigned)k >> LOG_L0;
            EXPECT(k + ((h == 0 ? 1 : 1 << (31 - __builtin_clz(h))) << LOG_L0) == q + L0 * c);
        }
    }
    // an entry that is not loaded is the first quarter's of its stage
    for (int c = 2; c < R; ++c)
        if (!quarter_loads(ENC_QUARTER, c)) {
            int top = 1;
            while (2 * top <= c) top *= 2;
            EXPECT(quarter_loads(ENC_QUARTER, c - top / 2));
        }
}

// The parts of a compact copy follow each other and fill it.
template <int LOG_NU, int LOG_E, int MODE, int PIPE, int LR0, int LR1, int LR2, bool MIXED = false> static void copy() {
    using PP = PassPlan<LOG_NU, LR0, LR1, LR2, 0>;
    constexpr int LAST = lds_twiddle_last_pass<LOG_NU, LOG_E, MODE, 0, PP, PIPE>();
    EXPECT(LAST >= 1);
    int at = 0;
    for (int p = 1; p <= LAST; ++p) {
        EXPECT(quarter_copy_offset<PP>(p) == at);
        at += (1 << (PP::log_l0(p) + PP::lr(p))) / 2;
    }
    constexpr bool COMPACT = compact_copy(ENC_QUARTER, PIPE, MODE, LOG_NU, MIXED);
    EXPECT(!compact_copy(ENC_TABLE, PIPE, MODE, LOG_NU, MIXED));
    constexpr int TE = lds_twiddle_entries<LOG_NU, LOG_E, MODE, 0, PP, PIPE, ENC_QUARTER, MIXED>();
    constexpr int PLAIN = lds_twiddle_entries<LOG_NU, LOG_E, MODE, 0, PP, PIPE, ENC_TABLE, MIXED>();
    EXPECT(TE % 2 == 0 && (COMPACT ? TE == at && TE <= PLAIN : TE == PLAIN));
}

// The split through the output: a column unit c of NUC points writes output k to
// c NUC + k of the transform, where row unit k reads its element c and writes its
// output c: the places k + c NUC, each with one owner.
static void through_output(int log_nuc, int log_nur) {
    const int nuc = 1 << log_nuc, nur = 1 << log_nur, n = nuc * nur;
    std::vector<int> owner(n, -1);
    for (int c = 0; c < nur; ++c)
        for (int k = 0; k < nuc; ++k) {
            const int place = (c << log_nuc) + k;            // the column kernel's store
            EXPECT(owner[place] == -1);
            owner[place] = k;                                 // the row unit that reads it
        }
    for (int k = 0; k < nuc; ++k)
        for (int e = 0; e < nur; ++e) EXPECT(owner[(e << log_nuc) + k] == k);   // strided loads and stores of row k
}

int main() {
    for (int64_t n = 1; n < 1100; ++n)
        for (int64_t bytes : {int64_t(1) << 20, kPlainOrderBytes, kPlainOrderBytes + 1}) {
            order<false>(n, bytes);
            order<true>(n, bytes);
        }
    order<false>(8192 + 77, 1 << 27);
    order<true>(8192 + 77, 1 << 27);
    slots<0, 1>(); slots<0, 5>(); slots<1, 2>(); slots<2, 3>(); slots<3, 4>(); slots<4, 4>(); slots<5, 5>();
    slots<6, 5>(); slots<9, 4>(); slots<8, 6>();
    copy<9, 3, MODE_SMALL, 3, 3, 3, 3>(); copy<11, 4, MODE_SMALL, 3, 3, 4, 4>(); copy<11, 4, MODE_SMALL, 3, 3, 4, 4, true>();
    copy<12, 4, MODE_SMALL, 5, 4, 4, 4>();
    copy<13, 5, MODE_SMALL, 3, 5, 4, 4>();
    copy<14, 5, MODE_SMALL, 5, 5, 5, 4>(); copy<16, 6, MODE_SMALL, 3, 6, 5, 5>(); copy<8, 4, MODE_COLS, 3, 4, 4, 0>();
    copy<9, 5, MODE_COLS, 3, 5, 4, 0>(); copy<10, 5, MODE_COLS, 3, 5, 5, 0>();
    for (int c = 7; c <= 8; ++c)
        for (int r = 6; r <= 8; ++r) through_output(c, r);
    for (int mode : {MODE_COLS, MODE_ROWS})
        for (int np = 2; np <= 3; ++np)
            for (int p = 0; p < np; ++p) {
                // strided accesses: the columns' loads, the rows' loads and stores
                using Out = GridGeoT<false, ENC_TABLE, 0, true>;
                const bool strided = mode == MODE_COLS ? p == 0 : (p == 0 || p == np - 1);
                const bool fast = mode == MODE_COLS ? unit_fast_pass<Out, MODE_COLS>(p, np) : unit_fast_pass<Out, MODE_ROWS>(p, np);
                if (p == 0 || p == np - 1) EXPECT(fast == strided);
            }
    std::printf("bad %d\n", bad);
    return bad != 0;
}
"""


def test_index_functions(tmp_path):
    try:
        hipcc = build._hipcc()
    except RuntimeError:
        pytest.skip("no hipcc")
    src, exe = tmp_path / "index.hip", tmp_path / "index"
    src.write_text(PROGRAM)
    r = subprocess.run([hipcc, "-x", "hip"] + [f for f in build.COMMON if f != "-O3"] + ["-O1"] + build.HIP_FLAGS +
                       ["-o", str(exe), str(src)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stdout
