"""Rows of the activations' copy that the tiles of the dense product fetch, 64 at a time: 192-row tiles
can end past the copy (padded to 256 rows), and no load may follow them there."""
from host_code import host_library


def test_no_band_leaves_the_padded_copy(tmp_path):
    lib = host_library(tmp_path, "bands", """
#include "common.hpp"
extern "C" int band_rows(int m0, int band, int padded) { return qalora::tile_band_rows(m0, band, padded); }
""")
    past = 0
    for M in list(range(129, 1600)) + [2048, 4096, 4097, 8191]:
        padded = (M + 255) // 256 * 256
        for m0 in range(0, M, 192):
            for band in range(3):
                off = lib.band_rows(m0, band, padded)
                assert 0 <= off and m0 + off + 64 <= padded
                if m0 + 64 * band < M:       # rows that are stored are the tile's own
                    assert off == 64 * band
                past += m0 + 64 * band + 64 > padded
    assert past > 0   # (the case exists: 193 rows, tiles to 384, a copy of 256)
