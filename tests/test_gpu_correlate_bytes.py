"""GPU parity of cpi_correlate on byte frames where its 256 x 256 tiles are
taken: frame counts around the 64- and 128-frame steps of its operand copies
(odd and even numbers of 64-frame blocks, one block only), values within and
above 127, whole and ragged tiles, and a workspace too small for rows in whole
cache lines.  Bit exact against the oracle."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import assert_bit_exact, log, oracle_in_layout, run_correlate

pytestmark = pytest.mark.gpu

PA, PB = 4000, 3050   # 16 x 12 tiles


def _case(n, pa, pb, top):
    rng = np.random.default_rng(n + 7 * top)
    fa = rng.integers(0, top, size=(n, pa), dtype=np.uint8)
    fb = rng.integers(0, top, size=(n, pb), dtype=np.uint8)
    return fa.reshape(-1), fb.reshape(-1)


@pytest.mark.parametrize("top", [128, 256])
@pytest.mark.parametrize("n", [64, 65, 128, 129, 192, 257])
def test_large_tiles(n, top):
    import paper_2407_20692_amd as cpi
    fa, fb = _case(n, PA, PB, top)
    log(f"case n={n} pa={PA} pb={PB} top={top}")
    ref = oracle.correlation(fa, fb, n, PA, PB, cpi.FRAMES_U8)
    for layout in (oracle.GAMMA_VIEW_MAJOR, oracle.GAMMA_PIXEL_MAJOR):
        got = run_correlate(cpi, fa, fb, n, PA, PB, cpi.FRAMES_U8, layout)
        assert_bit_exact(got, oracle_in_layout(ref, layout))


@pytest.mark.parametrize("n", [130, 300])
def test_workspace_without_line_rows(n):
    """A workspace a little below the reported size: the call stays accepted."""
    import torch
    import paper_2407_20692_amd as cpi
    pa, pb = 300, 140
    fa, fb = _case(n, pa, pb, 256)
    ref = oracle.correlation(fa, fb, n, pa, pb, cpi.FRAMES_U8)
    want = oracle_in_layout(ref, oracle.GAMMA_VIEW_MAJOR)["gamma"]
    need = cpi.correlate_workspace_size(n, pa, pb, cpi.FRAMES_U8)
    da, db = torch.from_numpy(fa).cuda(), torch.from_numpy(fb).cuda()
    for ws in (need, need - 256):
        log(f"case n={n} pa={pa} pb={pb} workspace={ws}")
        g = torch.empty(pa * pb, dtype=torch.float64, device="cuda")
        cpi.correlate(da, db, n, pa, pb, cpi.FRAMES_U8, cpi.GAMMA_VIEW_MAJOR, gamma=g,
                      workspace=cpi.alloc_workspace(ws))
        assert np.array_equal(g.cpu().numpy().view(np.int64), want.view(np.int64))
