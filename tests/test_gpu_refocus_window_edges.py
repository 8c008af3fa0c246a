"""GPU parity of the register-window x pass of the row-lane refocus at the
edges of its split, on stacks above the size that is gathered directly: 64-row
units (one row less, exact, one more, several), views of fewer than 16 rows,
view rows that start at any multiple of 4 bytes, 16-pair chunks that fall outside
the view, windows of which the LDS holds three, two or one over as many views,
fewer and more, plane counts around its groups and above one chunk.  Graded
like every refocus by max |I_gpu - I_oracle| / max |I_oracle| <= 1e-5 per plane,
on a seeded random FP32 Gamma; and equal bit for bit to the LDS-tap x pass, whose
sums run in the same order (the gathers' and the column-sum kernel's do not).
Which kernels ran is read from a trace; test_host_window checks the cases' plans."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import log
from tests.test_gpu_refocus import _run, assert_r12
from tests.test_gpu_refocus_rows import ROWS_SHAPES, _tiled
from tests.test_gpu_refocus_window import _geo

pytestmark = pytest.mark.gpu

CASES = [
    (_geo(65, 63, 9, 16), np.linspace(0.5, 1.5, 33)),
    (_geo(101, 64, 17, 10), np.linspace(0.8, 1.2, 17)),
    (_geo(150, 65, 11, 12, 131, 70), np.linspace(0.8, 1.2, 16)),
    (_geo(67, 129, 12, 27, 67, 100), np.linspace(0.95, 1.05, 9)),
    (_geo(256, 200, 3, 8), np.linspace(0.5, 1.5, 128)[:20]),
    (_geo(255, 130, 4, 3, 300, 140), np.linspace(1.3, 1.5, 40)),
    (_geo(128, 127, 33, 33), np.array([1.0])),
    (_geo(256, 8, 18, 30), np.linspace(0.9, 1.1, 20)),
    (_geo(129, 2, 80, 65), np.linspace(0.8, 1.2, 16)),
    (_geo(68, 17, 13, 5), np.linspace(0.7, 1.3, 300)),
    # planes whose samples leave the view on most columns and rows
    (oracle.Geometry(96, 80, 12, 12, 10.0, 10.0, 47.5, 39.5, 5.5, 5.5, 96, 80),
     np.linspace(0.5, 0.6, 18)),
] + [(_geo(128, 66, wb, hb), np.linspace(lo, hi, 4))
     for wb, hb in [(1, 500), (2, 250), (3, 170), (8, 64)]
     for lo, hi in [(0.5, 0.52), (0.8, 0.82), (0.97, 1.03)]]

# plane sets too spread for the window's registers, not for the LDS-tap x pass
WIDE = [
    (_geo(128, 70, 24, 20), np.array([0.62, 0.70, 0.78, 0.90])),
    (_geo(100, 130, 20, 30), np.array([1.2, 0.82, 1.1, 1.0, 0.95])),
]


def _launched(fn):
    """Names of the kernels that fn launches."""
    import torch
    from torch.profiler import ProfilerActivity, profile
    with profile(activities=[ProfilerActivity.CUDA]) as p:
        fn()
        torch.cuda.synchronize()
    return " ".join(e.key for e in p.key_averages())


def _case(i, seed, g, al):
    import paper_2407_20692_amd as cpi
    rng = np.random.default_rng(seed + i)
    gam32 = rng.standard_normal((g.hb * g.wb, g.ha * g.wa)).astype(np.float32)
    want = oracle.refocus(gam32.astype(np.float64), g, al)
    log(f"case {i}: {g}, {len(al)} planes")
    got = _run(cpi, cpi.refocus, gam32, g, al)
    assert_r12(got, want, i)
    assert np.array_equal(got, _run(cpi, cpi.refocus, gam32, g, al)), i
    same = 0
    for shape in ROWS_SHAPES:
        try:
            taps = _run(cpi, _tiled(cpi, shape + (1, cpi.REFOCUS_VIEW_ROWS, 0)), gam32, g, al)
        except cpi.CpiError as e:
            assert e.status == 2, e   # CPI_ERR_UNSUPPORTED
            continue
        assert np.array_equal(got, taps), (i, shape)
        same += 1
    return same


@pytest.mark.parametrize("i", range(len(CASES)))
def test_window_edges(i):
    _case(i, 980, *CASES[i])


@pytest.mark.parametrize("i", range(len(WIDE)))
def test_wider_windows(i):
    assert _case(i, 1010, *WIDE[i])


def test_kernels_launched():
    """cpi_refocus takes the register-window pass where it fits, else the LDS-tap
    pass; an explicit row-lane shape runs the LDS-tap pass as named."""
    import paper_2407_20692_amd as cpi
    rng = np.random.default_rng(1)
    for g, al, kernel in [CASES[1] + ("k_ref_window<",), WIDE[0] + ("k_ref_rows<",)]:
        gam32 = rng.standard_normal((g.hb * g.wb, g.ha * g.wa)).astype(np.float32)
        names = _launched(lambda: _run(cpi, cpi.refocus, gam32, g, al))
        assert kernel in names, names
        for na, xr in ROWS_SHAPES:
            fn = _tiled(cpi, (na, xr, 1, cpi.REFOCUS_VIEW_ROWS, 0))
            names = _launched(lambda: _run(cpi, fn, gam32, g, al))
            assert f"k_ref_rows<{na}, {xr}, " in names and "k_ref_window" not in names, names
