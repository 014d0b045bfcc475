"""The RGB stem with ReLU and its 3x3 / 2 max-pool in one pass, bit for bit
against the unfused stem's output pooled on the host: column blocks of 7
pooled pixels (a ragged last one, one block, the widest rows), every padding
(even ones start a lane's pixels on a whole word), one image cut into several
ranges of rows, more waves than the chip holds, an odd number of stem rows,
and infinities next to the padding."""

import numpy as np
import pytest
import torch

from workloads.configs import to_bf16_bits

pytestmark = pytest.mark.gpu

CASES = [
    # n, H, W, pad
    (1, 224, 224, 3),     # 8 column blocks, 14 ranges of 4 pooled rows
    (3, 7, 8, 3),         # 4 x 4 stem pixels, one block
    (2, 9, 16, 0),        # pad 0: 2 x 5 stem pixels
    (2, 61, 40, 1),       # odd rows of stem pixels
    (5, 40, 56, 2),       # 14 pooled columns: two whole blocks
    (2, 33, 64, 3),       # 16 pooled columns: a block of two
    (300, 30, 224, 3),    # more units than waves in flight
    (257, 8, 8, 3),
]


@pytest.mark.parametrize("special", [False, True], ids=["normal", "inf"])
@pytest.mark.parametrize("case", CASES, ids=str)
def test_stem_pool(case, special):
    from paper_2307_04963_amd import runtime
    n, H, W, pad = case
    rng = np.random.default_rng(H * W + n)
    x = torch.from_numpy(rng.standard_normal((n, H, W, 3)).astype(np.float32)).bfloat16()
    if special:      # the window's eighth slot and the padding must not turn them into NaN
        x[:, 0, 0], x[:, H - 1, W - 1], x[:, H // 2, W - 1] = float("inf"), float("inf"), float("-inf")
    w = rng.uniform(-0.2, 0.2, (64, 7, 7, 3)).astype(np.float32)
    if special:
        w = np.abs(w)
    packed = torch.from_numpy(runtime.pack_conv_weights(to_bf16_bits(w)).view(np.int16)).cuda()
    sc, sh = (torch.from_numpy(rng.uniform(lo, hi, 64).astype(np.float32)).cuda() for lo, hi in ((0.5, 1.5), (-0.3, 0.3)))
    xt = x.cuda()
    got = runtime.conv_maxpool(xt, packed, 64, 7, 2, pad, sc, sh).float().cpu()
    plain = runtime.conv(xt, packed, 64, 7, 2, pad, sc, sh, None, 1).float().cpu()
    want = torch.nn.functional.max_pool2d(plain.permute(0, 3, 1, 2), 3, 2, 1).permute(0, 2, 3, 1)
    assert not torch.isnan(got).any()
    assert torch.equal(got, want)
