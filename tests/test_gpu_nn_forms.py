"""Every kernel a convolution may take, at the sizes where the choice changes:
all sum in the same order, so the results are the same bits as from the kernel
that serves unaligned outputs (checked against FP64 elsewhere)."""
import pytest
import torch

from paper_2108_08591_amd import nn

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# (B, H, W, c1, c2, cout) on either side of the lines of nn_rules.h
SHAPES = [(1, 640, 128, 128, 0, 128), (1, 641, 128, 64, 64, 128), (1, 769, 128, 128, 0, 128), (1, 1280, 128, 96, 32, 128),
          (1, 511, 128, 288, 0, 128), (1, 512, 128, 256, 32, 128), (1, 768, 128, 64, 0, 128), (1, 1281, 128, 64, 0, 128),
          (1, 192, 128, 128, 0, 128), (1, 193, 128, 128, 0, 128), (1, 1280, 128, 128, 0, 64), (1, 1281, 128, 96, 32, 64),
          (1, 384, 128, 288, 0, 64), (1, 385, 128, 288, 0, 64), (1, 513, 128, 288, 0, 64), (1, 384, 128, 64, 0, 64),
          (3, 129, 127, 64, 0, 192), (1, 2047, 128, 96, 0, 32), (1, 2048, 128, 64, 32, 32), (1, 383, 128, 384, 0, 128),
          (5, 77, 91, 64, 0, 96), (2, 45, 67, 32, 0, 384), (9, 100, 120, 32, 0, 64), (33, 17, 129, 32, 0, 64)]


@pytest.mark.parametrize("shape", SHAPES)
def test_same_bits_as_the_unaligned_kernel(shape):
    B, H, W, c1, c2, co = shape
    print(f"[nn] forms {shape}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(sum(shape))

    def bf(*s):
        return torch.randn(s, generator=g, device=DEV).to(torch.bfloat16).view(torch.int16)

    x1, x2 = bf(B, H, W, c1), bf(B, H, W, c2) if c2 else None
    w, mask = bf(co, 9, c1 + c2), bf(B, H, W, co)
    bias = torch.linspace(-1, 1, co, device=DEV)
    n = B * H * W * co
    for relu, m, b in ((True, None, bias), (False, mask, None), (True, mask, bias), (False, None, None)):
        y = nn.bf16_empty((B, H, W, co), DEV)
        nn.conv_fwd(x1, x2, w, b, relu, mask=m, out_bf16=y)
        off = nn.bf16_empty((n + 8,), DEV)[1:1 + n].view(B, H, W, co)
        nn.conv_fwd(x1, x2, w, b, relu, mask=m, out_bf16=off)
        assert torch.equal(y, off)
        yf = torch.empty(B, H, W, co, device=DEV)
        nn.conv_fwd(x1, x2, w, b, relu, mask=m, out_f32=yf)
        off = torch.empty(n + 8, device=DEV)[1:1 + n].view(B, H, W, co)
        nn.conv_fwd(x1, x2, w, b, relu, mask=m, out_f32=off)
        assert torch.equal(yf, off)
