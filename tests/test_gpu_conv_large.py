"""Layers on inputs of 2^31 bytes and more (bf16 tensors may have up to 2^31 - 1
elements): rows on both sides of the 2^31st byte, the first rows of the image
after one that ends there, and the last rows, bit for bit against the same rows
run as an image of their own (a row's sums do not depend on the image's size)."""

import numpy as np
import pytest
import torch

from workloads.configs import to_bf16_bits

pytestmark = pytest.mark.gpu

CASES = [
    # n, H, cin, cout, k, stride; 64 pixels wide, so a row of 128 channels is 2^14 bytes
    (1, 140000, 128, 64, 3, 1),      # one image past 2^31 bytes: the 3x3 kernel on linear pixel tiles
    (2, 131071, 128, 64, 3, 1),      # a tile that starts in an image just below 2^31 bytes and ends in the next
    (1, 140000, 128, 64, 1, 1),      # the implicit GEMM, with addresses per lane from 2^31 bytes on
    (1, 140000, 128, 128, 3, 2),
]


@pytest.mark.parametrize("case", CASES, ids=str)
def test_conv_past_2_31_bytes(case):
    from paper_2307_04963_amd import runtime
    n, H, cin, cout, k, stride = case
    W, pad = 64, k // 2
    g = torch.Generator(device="cuda").manual_seed(H + k)
    x = torch.empty((n, H, W, cin), dtype=torch.bfloat16, device="cuda").normal_(generator=g)
    assert x.numel() * 2 > 2 ** 31
    w = np.random.default_rng(H).uniform(-0.05, 0.05, (cout, k, k, cin)).astype(np.float32)
    packed = torch.from_numpy(runtime.pack_conv_weights(to_bf16_bits(w)).view(np.int16)).cuda()
    y = runtime.conv(x, packed, cout, k, stride, pad)
    Ho = y.shape[1]
    row = 2 ** 31 // (W * cin * 2)   # image rows before the 2^31st byte, of all images
    at = {0, max(0, (row % H) // stride - 16), max(0, Ho - 32)}
    for i in range(n):
        for r0 in sorted(at):
            r1 = min(Ho, r0 + 32)
            # the input rows of output rows r0 .. r1 - 1, and 2 pad further ones whose outputs are not compared
            h0 = max(0, r0 * stride - stride * pad)
            part = x[i:i + 1, h0:min(H, r1 * stride + stride * pad)].contiguous()
            want = runtime.conv(part, packed, cout, k, stride, pad)[0, r0 - h0 // stride:][:r1 - r0]
            got = y[i, r0:r1]
            assert got.abs().sum() > 0
            assert torch.equal(got.view(torch.int16), want.view(torch.int16)), f"image {i}, rows {r0} to {r1 - 1}"
