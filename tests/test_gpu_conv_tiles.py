"""The 3x3 kernel on linear pixel tiles (stride 1, Cin and Cout multiples of
64) through dycl_op_conv, at the geometries where its tiles can go wrong:
tiles that cross rows and images, a ragged last tile, images of two pixels'
width, of two rows, and as wide as the patch allows, several input chunks,
and each of its three tile sizes; against the oracle's convolution with the
bound of test_gpu_conv (fp32 accumulation, one rounding to bf16)."""

import pytest

from tests.test_gpu_conv import _case

pytestmark = pytest.mark.gpu

CASES = [
    # n, H, W, cin, cout, k, stride, pad, residual, act
    (201, 12, 12, 64, 128, 3, 1, 1, False, 1),   # 128 x 128 tiles: every tile crosses rows, most an image
    (31, 28, 29, 64, 128, 3, 1, 1, True, 1),     # odd width, ragged last tile
    (127, 14, 14, 128, 128, 3, 1, 1, True, 2),   # two input chunks, GELU
    (125, 5, 5, 64, 1024, 3, 1, 1, False, 0),    # five images per tile, eight channel tiles
    (61, 14, 14, 64, 512, 3, 1, 1, True, 1),     # four channel tiles, ragged last tile
    (107, 14, 14, 256, 256, 3, 1, 1, True, 1),   # two channel tiles, four input chunks
    (100, 5, 5, 64, 1024, 3, 1, 1, False, 0),    # 128 x 64 tiles: sixteen channel tiles
    (9, 56, 56, 64, 128, 3, 1, 1, True, 1),      # wide images
    (3, 6, 79, 64, 128, 3, 1, 1, False, 1),      # the widest image a tile's patch holds
    (170, 14, 14, 128, 64, 3, 1, 1, False, 1),   # 64 output channels
    (1, 5, 5, 64, 128, 3, 1, 1, True, 1),        # 64 x 64 tiles: one tile, 25 of 64 pixels
    (3, 3, 43, 64, 128, 3, 1, 1, False, 1),
    (5, 2, 65, 64, 64, 3, 1, 1, False, 1),       # 64 -> 64 channels on few pixels: 128 x 64 tiles
    (6, 56, 56, 64, 64, 3, 1, 1, True, 1),       # 64 x 64 tiles
    (257, 11, 11, 64, 64, 3, 1, 1, True, 2),     # 64 x 64 tiles, 243 of 128 x 64
    (275, 11, 11, 64, 64, 3, 1, 1, True, 2),     # 128 x 64 tiles, 260
    (512, 8, 16, 64, 64, 3, 1, 1, True, 1),      # the last tile count they take
    (513, 8, 16, 64, 64, 3, 1, 1, True, 1),      # one more: the register-weight kernel
    (2, 5, 90, 64, 64, 3, 1, 1, False, 1),       # too wide for a patch: the register-weight kernel
    (5, 2, 65, 128, 64, 3, 1, 1, False, 1),      # two rows per image
    (4, 70, 2, 64, 128, 3, 1, 1, True, 1),       # two pixels per row
    (13, 7, 7, 256, 128, 3, 1, 1, True, 0),      # four input chunks
    (2, 3, 80, 64, 128, 3, 1, 1, False, 1),      # one pixel too wide: the implicit GEMM
    (300, 1, 1, 64, 128, 3, 1, 1, False, 1),     # 1 x 1 images: the implicit GEMM
    (13, 56, 56, 64, 128, 3, 1, 1, True, 1),     # wide images, 64 input channels, 638 tiles of 128 x 64
    (14, 56, 56, 64, 128, 3, 1, 1, True, 2),     # ... 686: the implicit GEMM
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "n{}_{}x{}_{}to{}".format(*c[:5]))
def test_conv3_tiles(case):
    _case(*case, seed=hash(case) % (2 ** 31))


@pytest.mark.parametrize("few,many,H,W,cout", [(20, 21, 56, 56, 64), (13, 14, 56, 56, 128), (3, 21, 37, 41, 512)])
def test_rows_do_not_depend_on_the_batch(few, many, H, W, cout):
    """64 input channels, on either side of the tile counts at which another
    kernel takes the layer: the first images' outputs are the same bits."""
    import numpy as np
    import torch
    from paper_2307_04963_amd import runtime
    from workloads.configs import to_bf16_bits
    rng = np.random.default_rng(many)
    x = torch.from_numpy(rng.standard_normal((many, H, W, 64)).astype(np.float32)).bfloat16().cuda()
    w = to_bf16_bits(rng.uniform(-0.1, 0.1, (cout, 3, 3, 64)).astype(np.float32))
    packed = torch.from_numpy(runtime.pack_conv_weights(w).view(np.int16)).cuda()
    a = runtime.conv(x, packed, cout, 3, 1, 1, act=2)[:few]
    b = runtime.conv(x[:few].contiguous(), packed, cout, 3, 1, 1, act=2)
    assert torch.equal(a.view(torch.int16), b.view(torch.int16))


@pytest.mark.parametrize("mode", ["sync", "device"])
def test_exit_after_a_wide_layer_does_not_depend_on_the_batch(mode):
    """An exit pools what a wide layer of 64 input channels wrote, on either
    side of the tile count at which another kernel takes the layer: the first
    images' logits are the same bits.  (600 classes: the exit's pooling is a
    launch of its own, or the layer's.)"""
    import json
    import numpy as np
    import torch
    from paper_2307_04963_amd import runtime
    from workloads.configs import to_bf16_bits
    rng = np.random.default_rng(3)
    blob = bytearray()

    def add(arr, bf16=False):
        blob.extend(b"\0" * ((-len(blob)) % 256))
        at = len(blob)
        arr = np.asarray(arr, np.float32)
        blob.extend((to_bf16_bits(arr) if bf16 else arr).tobytes())
        return at

    spec = {"version": 1, "dtype": "bf16", "input": {"name": "x", "shape": [56, 56, 64]}, "n_out": 600,
            "nodes": [{"op": "conv", "src": "x", "dst": "y", "k": 3, "stride": 1, "pad": 1, "cout": 128, "act": "relu",
                       "w": {"off": add(rng.uniform(-0.1, 0.1, (128, 3, 3, 64)), True)}, "scale": add(np.ones(128)),
                       "shift": add(np.zeros(128))},
                      {"op": "exit", "src": "y", "w": add(rng.uniform(-1, 1, (600, 128))), "b": add(np.zeros(600)),
                       "ncls": 600, "index": 0, "final": True}]}
    plan = runtime.Plan(json.dumps(spec), bytes(blob), 14)
    plan.set_host_mode(mode)
    x = torch.from_numpy(rng.standard_normal((14, 56, 56, 64)).astype(np.float32)).bfloat16().cuda()

    def run(n):
        logits, rec, _ = plan.outputs(n)
        plan.run(x[:n].contiguous(), None, logits, rec)
        torch.cuda.synchronize()
        return logits.clone()

    many = run(14)
    for n in (1, 13):
        assert torch.equal(run(n), many[:n])
    plan.close()
