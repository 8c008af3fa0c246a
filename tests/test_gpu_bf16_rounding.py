"""Float32 to bfloat16 as the denoiser's kernels round: every one of the 2^32 bit
patterns through the weight packing, against (u + 0x7FFF + (u >> 16 & 1)) >> 16, and
for NaN u >> 16 with the quiet bit set."""
import pytest

from tests.gpu_util import dev, log
from tests.test_gpu_denoiser import nn  # noqa: F401

pytestmark = pytest.mark.gpu


def test_every_float(nn):  # noqa: F811
    import torch
    n = 1 << 26
    low = torch.arange(n, dtype=torch.int32, device=dev())
    for k in range(64):
        u = low + torch.tensor((k << 26) - (1 << 32 if k >= 32 else 0), dtype=torch.int32,
                               device=dev())
        w, _ = nn.pack_weights(u.view(torch.float32).view(n // 32, 1, 1, 32), transposed=False)
        got = w.view(-1).view(torch.int16)
        top = u >> 16
        want = (u + 0x7FFF + (top & 1)) >> 16
        nan = (u & 0x7FFFFFFF) > 0x7F800000
        want = torch.where(nan, top | 0x40, want).to(torch.int16)
        assert torch.equal(got, want), k
    log("case bf16 rounding: 2^32 patterns")
