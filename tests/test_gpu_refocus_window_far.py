"""GPU parity of the register-window refocus where a work-group stages nine
16-column blocks and a wave's window starts past the eighth: two clusters of
planes, in order and not, a crop of a wide view, and both plane-group sizes.
Sizes are above the small stacks that are gathered directly.  Graded like every
refocus by max |I_gpu - I_oracle| / max |I_oracle| <= 1e-5 per plane, on a seeded
random FP32 Gamma."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import log
from tests.test_gpu_refocus import _run, assert_r12
from tests.test_gpu_refocus_window import _geo

pytestmark = pytest.mark.gpu


def _clusters(a, b, step, each):
    return np.concatenate([a + step * np.arange(each), b + step * np.arange(each)])


CASES = [
    (_geo(160, 40, 48, 12), _clusters(0.3, 1.4, 0.004, 4)),
    (_geo(160, 40, 48, 12), np.array([0.300, 0.304, 0.308, 0.312, 1.412, 1.400, 1.408, 1.404])),
    (_geo(256, 100, 29, 29, 32, 100), _clusters(0.53, 1.06, 0.004, 4)),
    (_geo(174, 64, 9, 12), _clusters(0.40, 1.82, 0.003, 8)),
]


@pytest.mark.parametrize("i", range(len(CASES)))
def test_far_windows(i):
    import paper_2407_20692_amd as cpi
    g, al = CASES[i]
    assert len(al) * g.out_w * g.out_h * g.wb * g.hb > 1 << 24
    rng = np.random.default_rng(960 + i)
    gam32 = rng.standard_normal((g.hb * g.wb, g.ha * g.wa)).astype(np.float32)
    want = oracle.refocus(gam32.astype(np.float64), g, al)
    log(f"case far window {i}: {g}, {len(al)} planes")
    got = _run(cpi, cpi.refocus, gam32, g, al)
    assert_r12(got, want, i)
    assert np.array_equal(got, _run(cpi, cpi.refocus, gam32, g, al)), i
