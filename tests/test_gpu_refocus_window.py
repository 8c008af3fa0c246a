"""GPU parity of the register-window x pass of the row-lane refocus at the
edges of its split: 64-row units (one row less, exact, one more, several
lens-plane rows per work-group), 16-column copies of views whose rows start
at any multiple of 4 bytes, 16-pair chunks that fall outside the view, and
plane counts around its groups of 4, 8 and 16.  Graded like every refocus by
max |I_gpu - I_oracle| / max |I_oracle| <= 1e-5 per plane, on a seeded random
FP32 Gamma."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import log
from tests.test_gpu_refocus import _run, assert_r12

pytestmark = pytest.mark.gpu


def _geo(wa, ha, wb, hb, out_w=None, out_h=None):
    return oracle.Geometry(wa, ha, wb, hb, wa / wb, ha / hb, (wa - 1) / 2, (ha - 1) / 2,
                           (wb - 1) / 2, (hb - 1) / 2, out_w or wa, out_h or ha)


CASES = [
    (_geo(65, 63, 9, 5), np.linspace(0.5, 1.5, 33)),
    (_geo(101, 64, 7, 9), np.linspace(0.8, 1.2, 17)),
    (_geo(150, 65, 4, 3, 131, 70), np.linspace(0.6, 1.4, 16)),
    (_geo(67, 129, 6, 11, 67, 100), np.linspace(0.95, 1.05, 9)),
    (_geo(256, 200, 3, 8), np.linspace(0.5, 1.5, 128)[:20]),
    (_geo(255, 130, 2, 2, 300, 140), np.linspace(1.3, 1.5, 40)),
    (_geo(128, 127, 1, 1), np.array([1.0])),
    (_geo(128, 2, 5, 3), np.linspace(0.7, 1.3, 5)),
    # planes whose samples leave the view on most columns and rows
    (oracle.Geometry(96, 80, 4, 4, 30.0, 30.0, 47.5, 39.5, 1.5, 1.5, 96, 80),
     np.linspace(0.5, 0.6, 18)),
]


@pytest.mark.parametrize("i", range(len(CASES)))
def test_window_edges(i):
    import paper_2407_20692_amd as cpi
    g, al = CASES[i]
    rng = np.random.default_rng(900 + i)
    gam32 = rng.standard_normal((g.hb * g.wb, g.ha * g.wa)).astype(np.float32)
    want = oracle.refocus(gam32.astype(np.float64), g, al)
    log(f"case window {i}: {g}, {len(al)} planes")
    got = _run(cpi, cpi.refocus, gam32, g, al)
    assert_r12(got, want, i)
    assert np.array_equal(got, _run(cpi, cpi.refocus, gam32, g, al)), i


@pytest.mark.parametrize("wb", [1, 2, 3, 8])
@pytest.mark.parametrize("lo,hi", [(0.5, 0.52), (0.8, 0.82), (0.97, 1.03)])
def test_window_stages(lo, hi, wb):
    """Windows of which the LDS holds three, two or one, over as many views,
    fewer and more."""
    import paper_2407_20692_amd as cpi
    g, al = _geo(128, 66, wb, 6), np.linspace(lo, hi, 4)
    rng = np.random.default_rng(int(1000 * lo) + wb)
    gam32 = rng.standard_normal((g.hb * g.wb, g.ha * g.wa)).astype(np.float32)
    want = oracle.refocus(gam32.astype(np.float64), g, al)
    log(f"case stages {lo} {hi} {wb}")
    got = _run(cpi, cpi.refocus, gam32, g, al)
    assert_r12(got, want, 0)
    assert np.array_equal(got, _run(cpi, cpi.refocus, gam32, g, al))
