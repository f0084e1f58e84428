"""The network's kernels at the sizes where their tiles, vectors and choices
of kernel end, against FP64.

Inputs are BF16 values, so a kernel differs from FP64 by its FP32
accumulation (bar 1e-5 relative, as for the other layer tests) and, for BF16
outputs, by one rounding (2^-8 relative)."""
import numpy as np
import pytest
import torch

from paper_2108_08591_amd import nn

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _bf(shape, seed, scale=1.0):
    g = torch.Generator().manual_seed(seed)
    v = (torch.randn(shape, generator=g) * scale).to(torch.bfloat16)
    return v.double(), v.view(torch.int16).to(DEV)


def _f(t):
    return t.view(torch.bfloat16).double().cpu()


def _rel(ref, got):
    return float(torch.linalg.vector_norm(ref - got.double().cpu()) / torch.linalg.vector_norm(ref).clamp_min(1e-300))


# tiles of 16 x 16 pixels: one, one less and one more row or column, single
# rows and columns; the last two take the kernel without pixel tiles (more
# than 512 blocks, padded more than 1.6 times)
CONV = [(1, 16, 16, 32, 0, 32), (2, 15, 17, 32, 32, 64), (1, 1, 40, 64, 0, 96), (2, 33, 1, 64, 64, 64),
        (1, 31, 65, 96, 32, 32), (3, 8, 9, 32, 96, 192), (41, 3, 200, 32, 0, 64), (33, 17, 129, 32, 32, 32),
        # runs of 128 pixels, 64 channels wide, and the widest blocks (384 input channels, 512 blocks)
        (2, 129, 128, 64, 0, 64), (1, 256, 257, 256, 128, 128)]


@pytest.mark.parametrize("shape", CONV)
def test_convolution(shape):
    B, H, W, c1, c2, co = shape
    print(f"[nn] tiles conv {shape}", flush=True)
    x1, d1 = _bf((B, H, W, c1), 1)
    x2, d2 = _bf((B, H, W, c2), 2) if c2 else (None, None)
    w, dw_ = _bf((co, 9, c1 + c2), 3, 0.1)
    dy, ddy = _bf((B, H, W, co), 4)
    m, dm = _bf((B, H, W, co), 5)
    bias = torch.linspace(-1, 1, co)
    x = (x1 if x2 is None else torch.cat([x1, x2], 3)).permute(0, 3, 1, 2)
    k = w.reshape(co, 3, 3, c1 + c2).permute(0, 3, 1, 2)
    ref = (torch.nn.functional.conv2d(x, k, bias.double(), padding=1)).permute(0, 2, 3, 1)
    yf = torch.full((B, H, W, co), float("nan"), device=DEV)
    nn.conv_fwd(d1, d2, dw_, bias.to(DEV), False, out_f32=yf)
    assert _rel(ref, yf) < 1e-5
    yb = nn.bf16_empty((B, H, W, co), DEV)
    nn.conv_fwd(d1, d2, dw_, bias.to(DEV), True, mask=dm, out_bf16=yb)
    want = ref.clamp_min(0) * (m > 0)
    assert _rel(want, _f(yb)) < 2.0 ** -8
    # an output 2 bytes off the alignment of the vector stores
    buf = torch.zeros(B * H * W * co + 8, dtype=torch.int16, device=DEV)
    off = buf[1:1 + B * H * W * co].view(B, H, W, co)
    nn.conv_fwd(d1, d2, dw_, bias.to(DEV), True, mask=dm, out_bf16=off)
    assert _rel(want, _f(off.contiguous())) < 2.0 ** -8
    assert int(buf[0]) == 0 and not buf[1 + B * H * W * co:].any()
    g = torch.full((co, 9, c1 + c2), float("nan"), device=DEV)
    gb = torch.full((co,), float("nan"), device=DEV)
    scratch = torch.empty(nn.wgrad_scratch_bytes(B, H, W, c1 + c2, co), dtype=torch.uint8, device=DEV)
    nn.conv_wgrad(d1, d2, ddy, g, gb, scratch)
    xp = torch.nn.functional.pad(x, (1, 1, 1, 1))
    dyf = dy.reshape(-1, co).t()
    gref = torch.stack([dyf @ xp[:, :, t // 3:t // 3 + H, t % 3:t % 3 + W].permute(0, 2, 3, 1).reshape(-1, c1 + c2)
                        for t in range(9)], 1)
    assert _rel(gref, g) < 1e-5
    assert _rel(dy.reshape(-1, co).sum(0), gb) < 1e-4       # a sum that cancels
    nn.conv_wgrad(d1, d2, ddy, g, None, scratch)
    assert _rel(gref, g) < 1e-5


@pytest.mark.parametrize("C,shift", [(8, 0), (24, 0), (12, 0), (1, 0), (8, 1)])
def test_pooling_upsampling_and_sum(C, shift):
    """Channels in vectors of 8 and one at a time, and pointers that allow no
    16-byte access: the same values."""
    B, H, W = 2, 6, 10

    def buf(shape):
        n = int(np.prod(shape))
        return torch.zeros(n + 8, dtype=torch.int16, device=DEV)[shift:shift + n].view(shape)

    def put(seed, shape):
        v, d = _bf(shape, seed)
        b = buf(shape)
        b.copy_(d)
        return v, b

    x, dx = put(1, (B, H, W, C))
    y, dy = put(2, (B, H, W, C))
    m, dm = put(3, (B, H, W, C))
    o = buf((B, H // 2, W // 2, C))
    nn.avgpool2(dx, o)
    s = x.reshape(B, H // 2, 2, W // 2, 2, C).sum((2, 4))
    assert _rel(0.25 * s, _f(o.contiguous())) < 2.0 ** -8
    o = buf((B, 2 * H, 2 * W, C))
    nn.upsample2(dx, o)
    assert torch.equal(_f(o.contiguous()), x.repeat_interleave(2, 1).repeat_interleave(2, 2))
    o = buf((B, H // 2, W // 2, C))
    nn.upsample2_bwd(dx, o)
    assert _rel(s, _f(o.contiguous())) < 2.0 ** -8
    o = buf((B, 2 * H, 2 * W, C))
    nn.avgpool2_bwd(dx, o)
    assert torch.equal(_f(o.contiguous()), (0.25 * x).repeat_interleave(2, 1).repeat_interleave(2, 2))
    for b, mask in ((dy, dm), (None, dm), (dy, None)):
        o = buf((B, H, W, C))
        nn.add(dx, b, mask, o)
        ref = (x + (y if b is not None else 0)) * ((m > 0) if mask is not None else 1)
        assert _rel(ref, _f(o.contiguous())) < 2.0 ** -8


@pytest.mark.parametrize("P,cin,cout", [(1, 32, 7), (255, 32, 8), (513, 32, 1), (1300, 32, 7), (257, 16, 7), (70, 24, 9)])
def test_head(P, cin, cout):
    x, dx_ = _bf((P, cin), 1)
    m, dm = _bf((P, cin), 2)
    g = torch.Generator().manual_seed(3)
    w, b, dy = (torch.randn(s, generator=g) for s in ((cout, cin), (cout,), (P, cout)))
    y = torch.full((P, cout), float("nan"), device=DEV)
    nn.head_fwd(dx_, w.to(DEV), b.to(DEV), y)
    assert _rel(x @ w.double().t() + b.double(), y) < 1e-5
    gx = nn.bf16_empty((P, cin), DEV)
    gw, gb = torch.empty(cout, cin, device=DEV), torch.empty(cout, device=DEV)
    scratch = torch.empty(nn.head_scratch_bytes(P, cin, cout), dtype=torch.uint8, device=DEV)
    if cin * cout + cout > 256:               # beyond what the backward call takes: refused
        with pytest.raises(RuntimeError):
            nn.head_bwd(dx_, dy.to(DEV), w.to(DEV), dm, gx, gw, gb, scratch)
        return
    nn.head_bwd(dx_, dy.to(DEV), w.to(DEV), dm, gx, gw, gb, scratch)
    assert _rel((dy.double() @ w.double()) * (m > 0), _f(gx)) < 2.0 ** -8
    assert _rel(dy.double().t() @ x, gw) < 1e-5
    assert _rel(dy.double().sum(0), gb) < 1e-5
