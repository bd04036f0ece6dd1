"""Addresses at which the error-compensated quantizer reads U, on the host: the kernel's own offset functions
over its schedule of loads.  The range check of a buffer load looks at the lane's offset alone, so a load
that passes it must be inside U whatever its row offset is; row offsets stay inside their block."""
import pytest

from host_code import host_library

BLOCK = 128


@pytest.fixture(scope="module")
def addr(tmp_path_factory):
    return host_library(tmp_path_factory.mktemp("addr"), "addr", """
#include "compensate_addr.hpp"
using namespace qalora;
extern "C" int block_rows(int d_in, int blk) { return comp_block_rows(d_in, blk); }
extern "C" int updates(int panels) { return comp_updates(panels); }
extern "C" unsigned update_lane(unsigned row_b, int nt, int r0, int n, int kb) { return comp_update_lane(row_b, nt, r0, n, kb); }
extern "C" unsigned update_row(unsigned row_b, int k, int q) { return comp_update_row(row_b, k, q); }
extern "C" unsigned walk_row(unsigned row_b, int rows, int s, int q) { return comp_walk_row(row_b, rows, s, q); }
""")


def update_block_reads(addr, d_in, blk, r0, nt):
    """First and last byte (relative to the block) of the updating loads of a block that pass the check."""
    row_b, size = 4 * d_in, addr.block_rows(d_in, blk) * 4 * d_in
    lanes = [addr.update_lane(row_b, nt, r0, n, kb) + 4 * h for kb in range(4) for n in range(16) for h in range(nt)]
    seen = [o for o in lanes if o < size]
    if not seen:
        return 0, 0
    return min(seen), max(seen) + addr.update_row(row_b, 7, 3) + 4


@pytest.mark.parametrize("d_in", [8, 16, 32, 64, 96, 120, 128, 136, 144, 208, 248, 256, 264, 384, 392, 512])
def test_updating_loads_stay_inside_u(addr, d_in):
    panels = (d_in + BLOCK - 1) // BLOCK
    if not addr.updates(panels):
        return
    for wave in range(3):
        nt = 3 if wave < 2 else 2
        for pn in range(panels):          # the panel being walked; the next one is brought up to date
            if pn + 1 >= panels and pn > 0:
                continue
            r0 = (pn + 1) * BLOCK + 48 * wave
            blocks = [(blk, r0) for blk in range(pn + 1)]        # what is loaded while panel pn + 1 is prepared
            blocks.append((0, r0 + BLOCK))                       # ... and ahead for the one after it
            for blk, r in blocks:
                lo, hi = update_block_reads(addr, d_in, blk, r, nt)
                assert lo >= 0 and blk * BLOCK * 4 * d_in + hi <= 4 * d_in * d_in


def test_one_panel_would_be_read_past_its_end(addr):
    # the reason for the rule: 64 rows of 64, read as if there were 128
    assert not addr.updates(1) and addr.updates(2)
    lo, hi = update_block_reads(addr, 64, 0, BLOCK, 3)
    assert hi > 4 * 64 * 64


@pytest.mark.parametrize("d_in", [8, 24, 120, 128, 136, 200, 264])
def test_walking_loads_stay_inside_the_panel(addr, d_in):
    row_b = 4 * d_in
    for pn in range((d_in + BLOCK - 1) // BLOCK):
        rows = addr.block_rows(d_in, pn)
        for s in range(8):
            for q in range(4):
                so = addr.walk_row(row_b, rows, s, q)
                assert so <= rows * row_b
                for kb in range(4):
                    row = 16 * s + 4 * q + kb
                    if row < rows:
                        assert so == (row - kb) * row_b    # existing rows are read where they are
                    for t in range(1, 8 - s):              # against the panel's later tiles
                        for n in (0, 15):
                            c = pn * BLOCK + 16 * (s + t) + n
                            if c < d_in:                   # (otherwise the lane's offset is past any buffer)
                                assert so + kb * row_b + 4 * c + 4 <= rows * row_b
