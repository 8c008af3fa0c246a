"""GPU parity of the ingest of frame rows that are no whole number of 4-byte
words: packed bits from 8 MiB of frames on (the tile kernel; below it the tail
kernel), one frame below, at and above, with rows of 4 to 7 bytes and a last
word of 1 to 3; bytes with rows of 1 to 9 pixels (loads of whole words from any
byte, and byte by byte below 4), and of 253 to 259, with counts above 127.
Small calls in both layouts, whose sums and outputs are stored in batches of 8.
Bit exact against the oracle."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import assert_bit_exact, log, oracle_in_layout, run_correlate

pytestmark = pytest.mark.gpu

LAYOUTS = (oracle.GAMMA_VIEW_MAJOR, oracle.GAMMA_PIXEL_MAJOR)


def _check(cpi, fa, fb, n, pa, pb, fmt, layouts=LAYOUTS):
    ref = oracle.correlation(fa, fb, n, pa, pb, fmt)
    for layout in layouts:
        got = run_correlate(cpi, fa, fb, n, pa, pb, fmt, layout)
        assert_bit_exact(got, oracle_in_layout(ref, layout))


# pixels of Da and Db; frames less the least for 8 MiB
@pytest.mark.parametrize("pa,pb,extra", [(8 * 41, 8 * 13 + 3, 0), (8 * 41, 8 * 13 + 3, -1),
                                         (1024 + 8 * 33, 8 * 6 + 1, 700), (8 * 4, 8 * 5, 0),
                                         (2048 + 8 * 2, 8 * 7, 1), (333, 32, 511)])
def test_bit_rows(pa, pb, extra):
    import paper_2407_20692_amd as cpi
    ra, rb = (pa + 7) // 8, (pb + 7) // 8
    n = (8 << 20) // (ra + rb) + extra
    rng = np.random.default_rng(pa + pb + extra)
    fa = rng.integers(0, 256, size=n * ra, dtype=np.uint8)
    fb = rng.integers(0, 256, size=n * rb, dtype=np.uint8)
    log(f"case bit rows pa={pa} pb={pb} n={n}")
    _check(cpi, fa, fb, n, pa, pb, cpi.FRAMES_BIT1, LAYOUTS[:1])


@pytest.mark.parametrize("pa,pb", [(1, 1), (2, 9), (3, 4), (4, 5), (5, 6), (6, 7), (7, 4), (9, 8),
                                   (253, 5), (254, 6), (255, 7), (257, 30), (258, 66), (259, 32)])
def test_byte_rows(pa, pb):
    import paper_2407_20692_amd as cpi
    for n in (63, 64, 130):
        rng = np.random.default_rng(pa * 100 + pb + n)
        fa = rng.integers(0, 256, size=(n, pa), dtype=np.uint8).reshape(-1)
        fb = rng.integers(0, 256, size=(n, pb), dtype=np.uint8).reshape(-1)
        log(f"case byte rows pa={pa} pb={pb} n={n}")
        _check(cpi, fa, fb, n, pa, pb, cpi.FRAMES_U8)


@pytest.mark.parametrize("pa,pb,n", [(30, 32, 68), (129, 65, 40), (127, 7, 513), (33, 191, 100),
                                     (1, 300, 77), (261, 1, 600)])
def test_small_bits(pa, pb, n):
    import paper_2407_20692_amd as cpi
    rng = np.random.default_rng(pa + pb + n)
    fa = rng.integers(0, 256, size=n * ((pa + 7) // 8), dtype=np.uint8)
    fb = rng.integers(0, 256, size=n * ((pb + 7) // 8), dtype=np.uint8)
    log(f"case small bits pa={pa} pb={pb} n={n}")
    _check(cpi, fa, fb, n, pa, pb, cpi.FRAMES_BIT1)
