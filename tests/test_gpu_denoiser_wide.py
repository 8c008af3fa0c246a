"""Denoiser gradients of very wide planes (up to 2^23 columns are accepted): 8
rows of columns just above where the LDS-staged kernels' 32-bit offsets end for
the first decoder layer (6 rows x W x 96 channels from 2^30 on), and of a
fifth of that.  The reference is the same network on the transposed planes with
transposed kernels, whose rows are short.  Both round the same sums to bfloat16,
which differ by float32 rounding only, so few elements round the other way;
bounds: a fifth of those of test_gpu_denoiser, where every element differs by
a bfloat16 rounding."""
import pytest

from tests.gpu_util import dev, log
from tests.test_gpu_denoiser import nn  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("w", [349536, 1864192])
def test_wide_gradients(nn, w):  # noqa: F811
    import torch
    assert (6 * w * 96 >= 1 << 30) == (w > 1000000)
    log(f"wide denoiser planes 8 x {w}")
    gen = torch.Generator(device=dev())
    gen.manual_seed(17)
    planes = torch.randn(1, 8, w, generator=gen, device=dev())
    targets = planes + 0.3 * torch.randn(1, 8, w, generator=gen, device=dev())
    net = nn.Denoiser(seed=6, device=dev())
    loss, grads = net.gradients(planes, targets)
    loss, grads = float(loss), grads.clone()
    flipped = net.params.clone()
    for L in nn.layers():
        a, _ = nn.layer_view(net.params, L)
        b, _ = nn.layer_view(flipped, L)
        b.copy_(a.transpose(1, 2))
    del net
    torch.cuda.empty_cache()
    ref = nn.Denoiser(params=flipped, device=dev())
    loss_ref, grads_ref = ref.gradients(planes.transpose(1, 2).contiguous(),
                                        targets.transpose(1, 2).contiguous())
    assert abs(loss - float(loss_ref)) <= 2e-3 * abs(loss)
    for L in nn.layers():
        gw, gb = nn.layer_view(grads, L)
        rw, rb = nn.layer_view(grads_ref, L)
        rw = rw.transpose(1, 2)
        ew = float((gw - rw).norm() / rw.norm())
        eb = float((gb - rb).norm() / rb.norm())
        log(f"  {L.name}: w {ew:.2e} b {eb:.2e}")
        assert ew <= 0.03 and eb <= 0.03, L.name
