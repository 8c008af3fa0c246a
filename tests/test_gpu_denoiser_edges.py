"""GPU parity of the LDS-staged 3x3 convolution and its weight gradient at the
edges of their tiles: one row and column less, exact and more, one to twelve
channel chunks, and one to many pixel blocks per work-group (three LDS stages).
The bounds of test_gpu_denoiser: a bfloat16 rounding of the result plus K float32
roundings of the absolute sum."""
import math

import numpy as np
import pytest

from oracle import denoiser as dn
from tests.gpu_util import dev, log
from tests.test_gpu_denoiser import bf16_tensor, host, nn, rand_bf16  # noqa: F401

pytestmark = pytest.mark.gpu

# b, h, w, cin, cout
CASES = [
    (40, 31, 47, 32, 32), (40, 33, 49, 32, 32), (30, 33, 31, 64, 64), (33, 31, 33, 96, 64),
    (70, 17, 15, 32, 64), (70, 15, 17, 384, 64), (9, 65, 63, 64, 32), (5, 66, 65, 32, 32),
    (5, 63, 129, 32, 64), (130, 8, 16, 64, 32),
]


@pytest.mark.parametrize("case", CASES, ids=[str(c) for c in CASES])
def test_conv3_edges(nn, case):  # noqa: F811
    import torch
    b, h, w, cin, cout = case
    log(f"conv3 edges {case}")
    rng = np.random.default_rng(b * h * w + cin)
    x = rand_bf16(rng, (b, h, w, cin))
    wt = (rng.standard_normal((cout, 3, 3, cin)) / math.sqrt(cin * 9)).astype(np.float32)
    wq = dn.round_bf16(wt)
    wf, _ = nn.pack_weights(torch.from_numpy(wt).to(dev()))
    of = torch.empty(b, h, w, cout, dtype=torch.float32, device=dev())
    nn.conv2d(bf16_tensor(x), wf, 3, cout, out_f32=of)
    ref, S = dn.conv2d(x, wq), dn.conv2d(np.abs(x), np.abs(wq))
    assert np.all(np.abs(host(of) - ref) <= 9 * cin * 2.0 ** -23 * S + 2.0 ** -24 * np.abs(ref))
    dy = rand_bf16(rng, (b, h, w, cout))
    ws = torch.empty(nn.conv2d_wgrad_workspace_size(b, h, w, cin, cout, 3), dtype=torch.uint8,
                     device=dev())
    dw = torch.zeros((cout, 3, 3, cin), dtype=torch.float32, device=dev())
    db = torch.zeros(cout, dtype=torch.float32, device=dev())
    nn.conv2d_wgrad(bf16_tensor(x), bf16_tensor(dy), 3, dw, db=db, workspace=ws)
    ref, S = dn.conv2d_grad_weight(x, dy, 3), dn.conv2d_grad_weight(np.abs(x), np.abs(dy), 3)
    m = b * h * w
    assert np.all(np.abs(host(dw) - ref) <= (m + 2) * 2.0 ** -23 * S)
    assert np.all(np.abs(host(db) - dn.bias_grad(dy)) <=
                  (m + 2) * 2.0 ** -23 * np.abs(dy).sum(axis=(0, 1, 2)))
