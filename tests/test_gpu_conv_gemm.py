"""The direct-to-LDS implicit GEMM through dycl_op_conv at each tile and stage
count that the dispatch chooses, with ragged row tiles, fewer K steps than
stages, channels that 64 does not divide (taps and sources per lane), and the
K split on few images; against the oracle's convolution with the bound of
test_gpu_conv (fp32 accumulation, one rounding to bf16)."""

import numpy as np
import pytest
import torch

from tests.test_gpu_conv import _case

pytestmark = pytest.mark.gpu

CASES = [
    # n, H, W, cin, cout, k, stride, pad, residual, act
    (105, 14, 14, 512, 256, 1, 1, 0, True, 1),     # 128 x 256 tiles, three stages
    (450, 7, 7, 64, 256, 1, 1, 0, False, 0),       # the same with one K step
    (450, 7, 7, 128, 256, 1, 1, 0, True, 2),       # two K steps, GELU
    (109, 14, 14, 128, 256, 3, 2, 1, False, 1),    # ... a strided 3x3 (42 tiles: 64 x 128)
    (420, 14, 14, 64, 256, 3, 2, 1, True, 1),      # ... and on 128 x 256 tiles
    (4003, 1, 1, 128, 1024, 1, 1, 0, False, 0),    # 128 x 128, three stages
    (4003, 1, 1, 192, 1024, 1, 1, 0, False, 2),
    (5003, 1, 1, 128, 896, 1, 1, 0, False, 1),     # 128 x 128, two stages
    (51, 7, 7, 512, 512, 1, 1, 0, True, 1),        # 64 x 128
    (11003, 1, 1, 64, 192, 1, 1, 0, True, 1),      # 128 x 64, three stages
    (65, 1, 1, 1024, 64, 1, 1, 0, False, 2),       # 64 x 64, 16 K steps, two row tiles
    (3, 5, 5, 64, 320, 1, 1, 0, True, 1),
    (301, 1, 1, 96, 64, 1, 1, 0, False, 1),        # 64 does not divide the channels
    (5, 9, 9, 32, 96, 3, 2, 1, True, 1),
    (7, 11, 11, 8, 40, 3, 2, 1, False, 2),         # 128 x 32 tiles, K = 72
    (521, 31, 32, 16, 32, 1, 2, 0, False, 1),      # ... and one stage: 128 x 32 tiles, one K step
    (521, 31, 32, 16, 24, 3, 2, 1, True, 1),       # three K steps, a ragged channel tile
    (521, 31, 32, 16, 32, 3, 2, 1, True, 2),       # GELU
    (521, 31, 32, 32, 64, 1, 2, 0, True, 0),       # 128 x 64 tiles
    (521, 31, 32, 16, 72, 3, 2, 1, False, 2),
    (521, 31, 32, 32, 64, 3, 2, 1, False, 1),      # five K steps: three stages
    (3, 7, 9, 16, 64, 7, 1, 3, False, 1),          # 7x7
    (60, 4, 4, 512, 512, 3, 1, 1, True, 1),        # K split on few images: 64 x 128 tiles
    (9, 8, 8, 512, 320, 3, 2, 1, False, 1),        # K split, 64-channel tiles
    # 1x1 on scalar addresses, one tile column's worth above and below
    (85, 14, 14, 256, 128, 1, 1, 0, True, 2),      # 64 x 64, two stages: short K
    (2100, 4, 4, 768, 64, 1, 1, 0, False, 1),      # ... and 64 channels
    (300, 14, 14, 128, 128, 1, 1, 0, True, 2),     # 128 x 64, one stage: one or two K steps
    (5, 56, 56, 256, 320, 1, 1, 0, False, 1),      # ... and other channel counts
    (33001, 1, 1, 128, 256, 1, 1, 0, False, 2),    # linear, 128 x 128 on one stage
    (301, 14, 14, 1024, 256, 1, 1, 0, True, 1),    # 128 x 256 on one stage, ragged rows
    (301, 14, 14, 1024, 256, 1, 1, 0, False, 2),
    (521, 16, 16, 64, 24, 1, 1, 0, True, 2),       # 128 x 32, two stages
    (521, 16, 16, 64, 24, 3, 1, 1, False, 1),
    (521, 31, 32, 64, 24, 3, 2, 1, False, 1),      # ... three: stride 2
    # addresses per lane
    (171, 14, 14, 96, 256, 1, 1, 0, True, 2),      # 128 x 128, one stage
    (42, 28, 28, 8, 256, 7, 1, 3, False, 1),       # ... 7x7
    (53, 14, 14, 160, 128, 1, 1, 0, True, 1),      # 64 x 128, three stages
    (171, 14, 14, 96, 128, 1, 1, 0, False, 0),     # ... two
    (13, 28, 28, 600, 320, 1, 1, 0, True, 1),      # ... three, a ragged channel tile, K = 600
    (19, 28, 28, 600, 320, 1, 1, 0, False, 2),     # ... two
    (85, 14, 14, 96, 96, 1, 1, 0, False, 1),       # 64 x 64, two stages
    (521, 16, 16, 240, 32, 1, 1, 0, True, 1),      # 128 x 32, two stages
    (3, 7, 7, 128, 512, 7, 1, 3, False, 1),        # K split: 64 x 128 tiles
    (90, 7, 7, 128, 512, 7, 1, 3, True, 2),        # ... 128 x 128, one stage
    (5, 7, 7, 128, 320, 7, 1, 3, False, 0),        # ... 64 x 64
    (57, 7, 7, 128, 320, 7, 1, 3, True, 1),        # ... 128 x 64
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "n{}_{}x{}_{}to{}_k{}s{}".format(*c[:7]))
def test_conv_gemm(case):
    _case(*case, seed=hash(case) % (2 ** 31))


def test_gelu_epilogue_matches_64_bits():
    """The GELU of the bf16 epilogues over its whole range, through a layer of
    identity weights: one rounding to bf16 (8 significant bits: half a unit in
    the last place is at most 2^-8 of the value) plus the epilogue's own error
    (5e-6 relative at |v| = 9 with every operation rounded to 32 bits, mostly the
    rounding of an exponent of 58; 0.5 v (1 + erff) has no digit left there)."""
    from paper_2307_04963_amd import runtime
    x = torch.linspace(-9, 9, 64 * 512).reshape(512, 1, 1, 64).bfloat16()
    w = torch.eye(64).reshape(64, 1, 1, 64).bfloat16()
    packed = torch.from_numpy(runtime.pack_conv_weights(w.view(torch.int16).numpy().view(np.uint16)).view(np.int16)).cuda()
    y = runtime.conv(x.cuda(), packed, 64, 1, 1, 0, act=2).cpu().double()
    v = x.double()
    ref = 0.5 * v * torch.erfc(-v / 2 ** 0.5)
    assert torch.all((y - ref).abs() <= ref.abs() * (2.0 ** -8 + 1e-5) + 1e-38)
    for edge, want in ((1e30, 1e30), (0.0, 0.0), (-1e30, 0.0)):
        z = torch.zeros((1, 1, 1, 64))
        z[..., 0] = edge
        got = runtime.conv(z.bfloat16().cuda(), packed, 64, 1, 1, 0, act=2).flatten()[0].item()
        assert abs(got - want) <= abs(want) * 2.0 ** -7
