"""GPU parity of cpi_correlate on packed-bit frames whose rows are no multiple of
4 bytes, with enough frames for the tile kernel: last words of 1, 2 and 3
bytes, the shortest rows it takes and shorter ones, rows past one 1024-pixel
tile, frame counts at and beside whole 512-frame tiles (the buffers end with the
last frame's last byte).  Bit exact against the oracle."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import assert_bit_exact, log, oracle_in_layout, run_correlate

pytestmark = pytest.mark.gpu

# pixels of Da and Db, frames
CASES = [(8 * 41, 8 * 13 + 3, 116512), (8 * 4, 8 * 5, 699392), (8 * 3, 8 * 5, 786944),
         (1024 + 8 * 33, 8 * 6 + 1, 38913), (2048 + 8 * 2, 8 * 7, 24063), (333, 32, 137216)]


@pytest.mark.parametrize("pa,pb,n", CASES)
def test_unaligned_rows(pa, pb, n):
    import paper_2407_20692_amd as cpi
    rng = np.random.default_rng(pa + pb)
    fa = rng.integers(0, 256, size=n * ((pa + 7) // 8), dtype=np.uint8)
    fb = rng.integers(0, 256, size=n * ((pb + 7) // 8), dtype=np.uint8)
    log(f"case rows pa={pa} pb={pb} n={n}")
    ref = oracle.correlation(fa, fb, n, pa, pb, cpi.FRAMES_BIT1)
    got = run_correlate(cpi, fa, fb, n, pa, pb, cpi.FRAMES_BIT1, oracle.GAMMA_VIEW_MAJOR)
    assert_bit_exact(got, oracle_in_layout(ref, oracle.GAMMA_VIEW_MAJOR))
