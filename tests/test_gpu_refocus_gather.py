"""GPU parity of the one-launch refocus of small stacks: fewer, as many and more
lens-plane columns than its 16 threads per pixel, output sizes that are no
multiple of its 16 pixels, samples outside the views, the most views its LDS
holds and one more (which the batched kernel takes), and the same in work and,
above that work, in planes.
Graded like every refocus by max |I_gpu - I_oracle| / max |I_oracle| <= 1e-5 per
plane, on a seeded random FP32 Gamma."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import log
from tests.test_gpu_refocus import _run, assert_r12
from tests.test_gpu_refocus_window import _geo

pytestmark = pytest.mark.gpu

CASES = [
    (_geo(2, 2, 1, 1), np.array([1.0])),
    (_geo(2, 3, 15, 2), np.array([0.5, 1.0, 1.5])),
    (_geo(5, 7, 16, 3, 9, 3), np.linspace(0.6, 1.4, 3)),
    (_geo(33, 17, 17, 5), np.linspace(0.5, 1.5, 5)),
    (_geo(31, 40, 3, 33), np.linspace(0.5, 1.5, 4)),
    (_geo(4, 4, 1023, 1), np.linspace(0.7, 1.3, 3)),
    (_geo(4, 4, 1023, 2), np.linspace(0.7, 1.3, 3)),
    (_geo(32, 32, 16, 16), np.linspace(0.5, 1.5, 64)),
    (_geo(32, 32, 16, 16), np.linspace(0.5, 1.5, 65)),
    # few planes at any size, with too wide a spread for the row-lane kernels,
    # and one more than those
    (_geo(128, 128, 32, 32), np.array([0.5, 1.5])),
    (_geo(40, 90, 33, 50), np.linspace(0.5, 1.5, 8)),
    (_geo(40, 90, 33, 50), np.linspace(0.5, 1.5, 9)),
    # planes whose samples leave the view on most columns and rows
    (oracle.Geometry(24, 20, 4, 4, 30.0, 30.0, 11.5, 9.5, 1.5, 1.5, 24, 20),
     np.linspace(0.5, 0.6, 6)),
]


@pytest.mark.parametrize("i", range(len(CASES)))
def test_gather_edges(i):
    import paper_2407_20692_amd as cpi
    g, al = CASES[i]
    rng = np.random.default_rng(700 + i)
    gam32 = rng.standard_normal((g.hb * g.wb, g.ha * g.wa)).astype(np.float32)
    want = oracle.refocus(gam32.astype(np.float64), g, al)
    log(f"case gather {i}: {g}, {len(al)} planes")
    got = _run(cpi, cpi.refocus, gam32, g, al)
    assert_r12(got, want, i)
    assert np.array_equal(got, _run(cpi, cpi.refocus, gam32, g, al)), i
