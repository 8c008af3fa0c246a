"""GPU parity of the 256 x 256 byte contraction in the modes that cpi_correlate
of few frames does not reach: running sums of a stream (int64 state; chunks of
odd and even numbers of 64-frame blocks, of one block, ragged, binary ones in
between), long frame runs at the fewer tiles that they need, and inputs of two and
three int32 passes, the last of two blocks.  Values above 127 are offset, pad
frames among them.  Bit exact against the oracle, or (long inputs) against
integers from exact float64 products."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import assert_bit_exact, dev, log, oracle_in_layout, run_correlate, to_dev
from tests.test_gpu_correlate_bytes import PA, PB
from tests.test_gpu_stream import _gamma

pytestmark = pytest.mark.gpu


def test_stream_chunks():
    import paper_2407_20692_amd as cpi
    sizes = [65, 128, 64, 130, 129, 192, 257, 1]
    n = sum(sizes)
    rng = np.random.default_rng(71)
    a = rng.integers(0, 256, size=(n, PA), dtype=np.uint8)
    b = rng.integers(0, 256, size=(n, PB), dtype=np.uint8)
    a[257:387] //= 128   # the fourth chunk is binary
    b[257:387] //= 128
    a[387:516] //= 2     # the fifth one needs no offset
    b[387:516] //= 2
    s = cpi.Stream(PA, PB, cpi.FRAMES_U8, max_chunk=257)
    lo = 0
    for k in sizes:
        log(f"case byte stream {PA} x {PB} chunk [{lo},{lo + k})")
        s.push(to_dev(a[lo:lo + k]), to_dev(b[lo:lo + k]), k)
        lo += k
        if k in (64, 192):
            ref = oracle.correlation(a[:lo], b[:lo], lo, PA, PB, oracle.FRAMES_U8)
            assert_bit_exact(_gamma(cpi, s, oracle.GAMMA_VIEW_MAJOR),
                             oracle_in_layout(ref, oracle.GAMMA_VIEW_MAJOR))
    ref = oracle.correlation(a, b, n, PA, PB, oracle.FRAMES_U8)
    for layout in (oracle.GAMMA_VIEW_MAJOR, oracle.GAMMA_PIXEL_MAJOR):
        assert_bit_exact(_gamma(cpi, s, layout), oracle_in_layout(ref, layout))
    s.close()


def test_long_rows_fewer_tiles():
    """144 tiles, taken from 64 blocks (4096 frames) on."""
    import paper_2407_20692_amd as cpi
    n, pa, pb = 4126, 4000, 2050
    rng = np.random.default_rng(72)
    fa = rng.integers(0, 256, size=(n, pa), dtype=np.uint8).reshape(-1)
    fb = rng.integers(0, 256, size=(n, pb), dtype=np.uint8).reshape(-1)
    log(f"case n={n} pa={pa} pb={pb}")
    ref = oracle.correlation(fa, fb, n, pa, pb, cpi.FRAMES_U8)
    got = run_correlate(cpi, fa, fb, n, pa, pb, cpi.FRAMES_U8, oracle.GAMMA_VIEW_MAJOR)
    assert_bit_exact(got, oracle_in_layout(ref, oracle.GAMMA_VIEW_MAJOR))


@pytest.mark.parametrize("n,pa,top", [(131008 + 65, 49150, 128), (2 * 131008 + 65, 49150, 256),
                                      (2 * 131008 + 4100, 32700, 256)])
def test_several_passes(n, pa, top):
    import torch
    import paper_2407_20692_amd as cpi
    pb = 200
    log(f"case n={n} pa={pa} pb={pb} top={top}")
    gen = torch.Generator(device=dev())
    gen.manual_seed(n)
    fa = torch.empty(n, pa, dtype=torch.uint8, device=dev())
    fb = torch.empty(n, pb, dtype=torch.uint8, device=dev())
    num = torch.zeros(pb, pa, dtype=torch.float64, device=dev())
    sa = torch.zeros(pa, dtype=torch.int64, device=dev())
    for i in range(0, n, 8192):
        x, y = fa[i:i + 8192], fb[i:i + 8192]
        x.random_(0, top, generator=gen)
        y.random_(0, top, generator=gen)
        num += y.double().t().contiguous() @ x.double()   # exact: sums below 2^53
        sa += x.sum(0, dtype=torch.int64)
    sb = fb.sum(0, dtype=torch.int64)
    want = (num.to(torch.int64) * n - sb[:, None] * sa[None]).view(-1)
    del num
    numer = torch.empty(pa * pb, dtype=torch.int64, device=dev())
    gamma = torch.empty(pa * pb, dtype=torch.float64, device=dev())
    ga, gb = torch.empty_like(sa), torch.empty_like(sb)
    cpi.correlate(fa.view(-1), fb.view(-1), n, pa, pb, cpi.FRAMES_U8, cpi.GAMMA_VIEW_MAJOR,
                  gamma=gamma, numer=numer, sum_a=ga, sum_b=gb)
    torch.cuda.synchronize()
    assert torch.equal(ga, sa) and torch.equal(gb, sb)
    assert torch.equal(numer, want)
    # (by numpy: torch divides by a number as a product with its reciprocal)
    quotient = want.cpu().numpy().astype(np.float64) / (float(n) * float(n))
    assert np.array_equal(gamma.cpu().numpy(), quotient)
