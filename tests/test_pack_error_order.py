"""Of several refused groups in a matrix the first one in the order of the entries is
reported: tile by tile, in a tile column by column, in a column row by row."""

import itertools

import numpy as np
import pytest

from paper_2607_02893_amd import vbq

CODE_RANGE, NONFINITE, SCALE_RANGE = 4, 5, 6


def _first(faults, R):
    return min(faults, key=lambda f: (f[0] // R, f[1], f[0]))[2]


# two faults each: rows and columns in either order, in one tile and in two, one of
# them a 1-bit mean that overflows fp16 (known only after other groups)
PLACES = [(0, 0), (0, 3), (3, 1), (5, 0), (5, 3), (15, 1), (16, 0), (17, 2), (30, 1)]


@pytest.mark.parametrize("threads", [1, 0])
@pytest.mark.parametrize("bits_of_wide", [1, 8])
def test_pack_reports_the_first_refused_group(threads, bits_of_wide):
    N, G, R = 31, 4, 16
    for a, b in itertools.permutations(PLACES, 2):
        if threads == 0 and a[0] // R != b[0] // R:
            continue  # tiles of several threads: whichever is met first
        W = np.ones((N, 64 * G), dtype=np.float32)
        bits = np.full((N, G), 2, dtype=np.uint8)
        W[a[0], 64 * a[1]:64 * a[1] + 64] = 1e8  # its scale overflows fp16 at every width
        bits[a] = bits_of_wide
        W[b[0], 64 * b[1] + 7] = np.nan
        with pytest.raises(vbq.VbqError) as e:
            vbq.pack(W, bits, tile_rows=R, chunk_groups=2, n_threads=threads)
        assert e.value.status == _first([(*a, SCALE_RANGE), (*b, NONFINITE)], R), (a, b)


def test_pack_codes_reports_the_first_refused_group():
    N, G, R = 31, 4, 16
    for a, b, c in itertools.permutations(PLACES, 3):
        q = np.ones((N, 64 * G), dtype=np.int8)
        s = np.full((N, G), 0x3C00, dtype=np.uint16)
        bits = np.full((N, G), 2, dtype=np.uint8)
        q[a[0], 64 * a[1] + 5] = 2
        s[b] = 0x7C00
        s[c] = 0xBC00
        with pytest.raises(vbq.VbqError) as e:
            vbq.pack_codes(q, s, bits, tile_rows=R, chunk_groups=2, n_threads=1)
        assert e.value.status == _first([(*a, CODE_RANGE), (*b, NONFINITE), (*c, SCALE_RANGE)], R), (a, b, c)
