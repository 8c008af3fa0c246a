"""GPU parity of cpi_correlate where its output tiles end: detector sizes one
below, at and one above the 128-wide tiles and their 64-row halves, aligned
and unaligned rows, both storage orders, for every operand encoding.  Bit
exact against the oracle."""
import numpy as np
import pytest

import oracle
from synth import pack_bits_lsb
from tests.gpu_util import assert_bit_exact, log, oracle_in_layout, run_correlate

pytestmark = pytest.mark.gpu

SIZES = [(127, 63), (128, 64), (129, 65), (131, 191), (132, 130), (36, 257), (260, 33)]


def _frames(kind, n, npix, rng):
    if kind == "bits" or kind == "binary":
        x = (rng.random((n, npix)) < 0.2).astype(np.uint8)
    else:
        x = rng.integers(0, 256 if kind == "large" else 40, size=(n, npix), dtype=np.uint8)
    return x


@pytest.mark.parametrize("layout", [oracle.GAMMA_VIEW_MAJOR, oracle.GAMMA_PIXEL_MAJOR])
@pytest.mark.parametrize("kind", ["bits", "binary", "counts", "large"])
@pytest.mark.parametrize("pa,pb", SIZES)
def test_tile_edges(pa, pb, kind, layout):
    import paper_2407_20692_amd as cpi
    for n in (65, 1100):
        rng = np.random.default_rng(1000 * pa + 10 * pb + n)
        fa, fb = _frames(kind, n, pa, rng), _frames(kind, n, pb, rng)
        fmt = cpi.FRAMES_BIT1 if kind == "bits" else cpi.FRAMES_U8
        if kind == "bits":
            fa, fb = pack_bits_lsb(fa), pack_bits_lsb(fb)
        fa = np.concatenate([fa.reshape(-1), np.zeros(16, np.uint8)])
        fb = np.concatenate([fb.reshape(-1), np.zeros(16, np.uint8)])
        log(f"case n={n} pa={pa} pb={pb} kind={kind} layout={layout}")
        ref = oracle.correlation(fa, fb, n, pa, pb, fmt)
        got = run_correlate(cpi, fa, fb, n, pa, pb, fmt, layout)
        assert_bit_exact(got, oracle_in_layout(ref, layout))
